// What is left of a call when its main kernel is done with its tiles: see ef_tile.h for the tile scheme.
#pragma once
#include "ef_tile.h"

namespace ef {

// How long a workgroup waits for partial sums that are sure to come.  Should one never show, the scale is a NaN rather than one
// formed from the last call's words.
constexpr int SURE_POLLS = 1 << 20;
__device__ __forceinline__ double sure_word(const unsigned long long *at, unsigned long long tag)
{
#pragma unroll 1
    for (int it = 0; it < SURE_POLLS; ++it) {
        const unsigned long long w = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((w >> 63) == tag) return __longlong_as_double((long long)(w & ~TAG_BIT));
        __builtin_amdgcn_s_sleep(8);
    }
    return __longlong_as_double(0x7ff8000000000000ll);
}

// Nothing that the call has made can be relied on: every scale of it becomes a NaN, which no result that is made from them hides.
__device__ __forceinline__ void spoil_call(const Layout &L, const ScratchRef &R)
{
#pragma unroll 1
    for (int w = 0; w < R.nsets; ++w)
#pragma unroll 1
        for (int64_t b = lane_id(); b < L.B; b += 64) R.scales[(int64_t)w * R.scales_stride + b] = __uint_as_float(0x7fc00000u);
}

// An entry that is there or on its way (one wavefront): its workgroup runs, and what it waits for is bounded.  Should it not come, a
// segment that nobody knows would keep p, and its block's scale not be written: the call is spoiled.  The entry stays, if it
// does come; it is of this call (parked_in), so no other call takes it.
__device__ __forceinline__ unsigned long long take_entry(unsigned long long *at, const Layout &L, const Scratch &X)
{
    const unsigned long long it = uniform_u64(await_parked([&] { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                                                           [] { __builtin_amdgcn_s_sleep(8); }, X.epoch, SURE_POLLS));
    if (!it)
        spoil_call(L, call_args().R);
    else if (lane_id() == 0)
        *at = 0ull;
    return it;
}

// A workgroup sees to its own parked segments, the last one to have begun to the `left` entries of others too, which are there or
// on their way.  Their blocks' partial sums are sure to come.  (Waits run out only where something else holds the GPU, so
// one wavefront for all of it is enough.)
__device__ __forceinline__ void end_left_over(unsigned left, const Scratch &X, SyncShared &S)
{
    const CallArgs &C = call_args();
    const Layout &L = C.L;
    const ScratchRef &R = C.R;
    const int lane = lane_id();
#pragma unroll 1
    for (unsigned i = 0; i < left + 2u; ++i) {
        const unsigned long long it = i < 2u ? uniform_u64(S.own[i]) : take_entry(R.parked + (i - 2u), L, X);
        if (!it) continue;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int set = parked_set(it), w = set - X.set_base;
        const int32_t tile = parked_tile(it);
        const int64_t b = parked_slot(it) ? L.tile_lb[tile] : L.tile_fb[tile], start = (int64_t)tile * TILE;
        const BlockSpan sp = block_span(L, b);
        // the order of gather_scale, which has four wavefronts
        const unsigned long long *part = set_part(X, L, set);
        const unsigned long long tag = set_tag(X, set);
        double total = 0.0;
#pragma unroll 1
        for (int q = 0; q < NWAVES; ++q) {
            double acc = 0.0;
#pragma unroll 1
            for (int t = 64 * q + lane; t < sp.n; t += THREADS) acc += sure_word(part + part_index(sp.t0 + t, sp), tag);
            total = q == 0 ? wave_sum(acc) : total + wave_sum(acc);
        }
        const float s = (float)(total / (double)(sp.be - sp.bs));
        if ((it & PARKED_FORMS) && lane == 0) post_scale(b, sp, s, L, X, set, R.scales + (int64_t)w * R.scales_stride);
        float *e = R.err + (int64_t)w * R.err_stride + start;
        const int lo = (int)max(sp.bs - start, (int64_t)0);
        const int hi = (int)min(sp.be - start, (int64_t)((it & PARKED_BOTH) ? 2 * TILE : TILE));
#pragma unroll 1
        for (int j = lo + lane; j < hi; j += 64) e[j] = residual(e[j], s);
    }
}

// End of a main kernel's workgroup.  left: what arrived() answered.
__device__ __forceinline__ void end_call(unsigned left, const ScratchRef &R, const Scratch &X, SyncShared &S)
{
    if (!X.ends) {
        snapshot_call(R);
    } else if (uniform_u32(threadIdx.x >> 6) == 0u) {
        const unsigned own = uniform_u32((unsigned)((S.own[0] | S.own[1]) >> 32));
        if (left | own) end_left_over(left, X, S);
    }
}

}  // namespace ef
