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

// An entry that is there or on its way (one wavefront): its workgroup runs, and what it waits for is bounded.  Should it not come, a
// segment that nobody knows keeps p, and its block's scale may not be written: 0, and see LOST.  The entry stays, if it
// does come; it is of this call (parked_in), so no other call takes it.
__device__ __forceinline__ unsigned long long take_entry(unsigned long long *at, const Scratch &X)
{
    const unsigned long long it = uniform_u64(await_parked([&] { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                                                           [] { __builtin_amdgcn_s_sleep(8); }, X.epoch, SURE_POLLS));
    if (it && lane_id() == 0) *at = 0ull;
    return it;
}

// e <- p - Delta over the elements [lo, hi) of a residual row whose p was parked (one wavefront).
__device__ __forceinline__ void residual_range(float *e, int64_t lo, int64_t hi, float s)
{
    const int lane = lane_id();
    const int64_t a = (lo + 3) & ~(int64_t)3, z = hi & ~(int64_t)3;     // whole groups of four
    if (a >= z) {
        if (lo + lane < hi) e[lo + lane] = residual(e[lo + lane], s);
        return;
    }
    // the other elements of the first and the last group may be another wavefront's
    if (lo + lane < a) e[lo + lane] = residual(e[lo + lane], s);
    if (z + lane < hi) e[z + lane] = residual(e[z + lane], s);
    constexpr int DEEP = 4;             // loads in flight a lane (eight: up to 18 spilled registers, 1654 us for end_call's 1740)
#pragma unroll 1
    for (int64_t j = a + 4 * lane; j < z; j += DEEP * 256) {
        float4 v[DEEP];
#pragma unroll
        for (int q = 0; q < DEEP; ++q) v[q] = *reinterpret_cast<const float4 *>(e + min(j + 256 * q, z - 4));
#pragma unroll
        for (int q = 0; q < DEEP; ++q) {
            residual4(v[q], s);
            if (j + 256 * q < z) *reinterpret_cast<float4 *>(e + j + 256 * q) = v[q];
        }
    }
}

// Finishes the segment of an entry, whose block's partial sums are sure to come (one wavefront).  In place of one that did not
// come, LOST: the first segment of the call's first set gets a NaN for its scale, which nothing that is made from the call hides.
constexpr unsigned long long LOST = 0ull;
__device__ __forceinline__ void finish_entry(unsigned long long it, const Layout &L, const Scratch &X, const ScratchRef &R)
{
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const int w = it == LOST ? 0 : parked_set(it) - X.set_base, set = X.set_base + w, lane = lane_id();
    const int32_t tile = parked_tile(it);
    const int64_t b = parked_slot(it) ? L.tile_lb[tile] : L.tile_fb[tile], start = (int64_t)tile * TILE;
    const BlockSpan sp = block_span(L, b);
    // a scale that has been posted saves a large block's sums
    unsigned long long posted = 0ull;
    if (sp.n > THREADS) posted = uniform_u64(__hip_atomic_load(ready_word(X, L, set, sp), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    float s = it == LOST ? __uint_as_float(0x7fc00000u) : __uint_as_float((unsigned)posted);
    if (it != LOST && (unsigned)(posted >> 32) != X.epoch) {
        // the order of gather_scale, which has four wavefronts
        const unsigned long long *part = set_part(X, L, set);
        const unsigned long long tag = set_tag(X, set);
        double acc[NWAVES] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int t = lane; t < sp.n; t += THREADS)
#pragma unroll
            for (int q = 0; q < NWAVES; ++q)
                if (t + 64 * q < sp.n) acc[q] += sure_word(part + part_index(sp.t0 + t + 64 * q, sp), tag);
        double total = wave_sum(acc[0]);
#pragma unroll
        for (int q = 1; q < NWAVES; ++q) total += wave_sum(acc[q]);
        s = (float)(total / (double)(sp.be - sp.bs));
    }
    if ((it == LOST || (it & PARKED_FORMS)) && lane == 0) post_scale(b, sp, s, L, X, set, R.scales + (int64_t)w * R.scales_stride);
    residual_range(R.err + (int64_t)w * R.err_stride, max(sp.bs, start), min(sp.be, start + ((it & PARKED_BOTH) ? 2 * TILE : TILE)), s);
}

// The entries of the call, as many as the last workgroup to begin has found (LEFT), are shared out a wavefront to each: between
// that one, the last ones of their groups that found some (arrived), and those whose own wait ran out when all had begun.
// All but the first may wait for LEFT, bounded, and go if it does not come.  (Figures at end_call.)
constexpr int HELP_POLLS = 1 << 16;
// own: the workgroup's own two; with_own: they are this wavefront's to see to.
__device__ __forceinline__ void finish_entries(const unsigned long long *own, bool with_own, const Scratch &call)
{
    const Layout &L = call_args().L;
    const ScratchRef &R = call_args().R;
    Scratch X = call;                   // what need not be kept from the kernel's start is read again
    X.part = R.part;
    X.ready = R.ready;
    X.set_base = R.set_base;
    unsigned n = 0u;
#pragma unroll 1
    for (int i = with_own ? 0 : 2;; ++i) {
        unsigned long long it;
        if (i < 2) {
            it = uniform_u64(own[i]);
        } else {
            if (i == 2)
#pragma unroll 1
                for (int q = 0; q < HELP_POLLS && !n; ++q) {
                    if (q) __builtin_amdgcn_s_sleep(8);
                    n = uniform_u32(__hip_atomic_load(arrive_word(X, LEFT), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
            unsigned k = 0u;
            if (n > 1u && lane_id() == 0) k = atomicAdd(arrive_word(X, TAKEN), 1u);
            k = uniform_u32(k);
            if (k + 1u >= n) return;
            it = take_entry(R.parked + k, X);
        }
        if (i >= 2 || it) finish_entry(it, L, X, R);
    }
}

// End of a main kernel's workgroup.  left: what arrived() answered.  A worker call whose every wait gives up, ended
// by k_tail / by one wavefront alone / as it is, us: ResNet-50 (6306 tiles) 924 / 179 386 / 1740, 2^26 elements in blocks of 2^20
// 2205 / 456 116 / 4182, 300 000 blocks of 33 774 / 10 281 / 633.  (Workgroups behind the tiles' for it, sixteen, 1223 at the first:
// their branch at every workgroup's start costs the ResNet-50's server call 1.1 of 42.5 us.)
__device__ __forceinline__ void end_call(unsigned left, const ScratchRef &R, const Scratch &X, SyncShared &S)
{
    if (!X.ends) {
        snapshot_call(R);
    } else if (uniform_u32(threadIdx.x >> 6) == 0u) {
        const unsigned own = uniform_u32((unsigned)((S.own[0] | S.own[1]) >> 32));
        if (left | own) finish_entries(S.own, true, X);
    }
}

}  // namespace ef
