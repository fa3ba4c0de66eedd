// Compressor-quality diagnostics of libef (Section 3.2 of arxiv 1905.10936): see ef_tile.h for the tile scheme.
#pragma once
#include "ef_tile.h"

namespace ef {

// ------------------------------------------------- compressor quality ---
//
// phi(v) = min_b ||v_Gb||_1^2 / (d_b ||v_Gb||_2^2) (Proposition 1) and
// delta(v) = ||v||_1^2 / (d ||v||_2^2) (non-block compressor, Eq. (1)), in
// fp64.  Per tile (a pass of its own over v, or
// inside the worker kernel on the p it has in registers anyway) the sums of |v| and v^2
// of the tile and of its open segments, and the ratios of the segments that
// close inside the tile; per crossing block the sums of its tiles' partials in
// a fixed order.  The minimum is taken with an integer atomic on the bits of
// the (non-negative) ratio, which does not depend on the order of arrival, in a word of the plan that is 1 between calls (the
// ratio of an all-zero block, which the compressor reproduces exactly): the last of a vector's workgroups in the second kernel
// writes it out and puts the 1 back.  (A kernel of its own that sets the word to 1 ahead of the two, as k_quality_reset does after a
// call that has failed between them: 6 vectors of 66 tiles 12.4 us, 12.1 without; ResNet-50, 4 vectors, 74.2 and 73.6.)

struct QualityArgs {
    const float *v;             // [n][stride]
    int64_t stride;
    double *tile_sums;          // [n][ntiles][2]   (sum |v|, sum v^2) of each tile
    double *part_sums;          // [n][2*ntiles][2] the same for each open segment (slot as in part_index)
    double *out;                // [n][2]           phi, delta
    unsigned long long *phi;    // [n]              bits of the smallest ratio so far, of 1.0 between calls
    unsigned *done;             // [n]              workgroups of k_quality_blocks that are through, 0 between calls
};

__device__ __forceinline__ void ratio_min(unsigned long long *phi_bits, double l1, double l2, int64_t db)
{
    if (l2 > 0.0) {
        const double ratio = l1 * l1 / ((double)db * l2);
        atomicMin(phi_bits, (unsigned long long)__double_as_longlong(ratio));
    }
}

// The words as they are between calls.
__global__ __launch_bounds__(THREADS) void k_quality_reset(unsigned long long *phi, unsigned *done, int n)
{
    for (int i = threadIdx.x; i < n; i += THREADS) {
        phi[i] = (unsigned long long)__double_as_longlong(1.0);
        done[i] = 0u;
    }
}

// The share of one tile of vector `vec` in phi and delta: a holds the tile's values (any sign; past
// the end of the vector 0).  Called by every thread of the workgroup; uses S.red, and for a tile
// where several blocks meet S.val and S.long_list as well (free again on return).
__device__ __forceinline__ void quality_of_tile(float4 (&a)[SUBROWS], const Layout &L, const QualityArgs &Q, int32_t tile,
                                                int vec, int n_valid, TileShared &S)
{
    __shared__ double seg_sum[2][2];            // [head, tail][l1, l2] of the open segments
    __shared__ unsigned long long tile_min;
    const int64_t tile_start = (int64_t)tile * TILE;
    const int32_t fb = L.tile_fb[tile], lb = L.tile_lb[tile];
    unsigned long long *phi_bits = Q.phi + vec;
    double l1 = 0.0, l2 = 0.0;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        a[k] = make_float4(fabsf(a[k].x), fabsf(a[k].y), fabsf(a[k].z), fabsf(a[k].w));
        const double x = a[k].x, y = a[k].y, z = a[k].z, w = a[k].w;
        l1 += (x + y) + (z + w);
        l2 += (x * x + y * y) + (z * z + w * w);
    }
    l1 = block_sum(l1, S.red);
    l2 = block_sum(l2, S.red);
    double *ts = Q.tile_sums + ((int64_t)vec * L.ntiles + tile) * 2;
    double *ps = Q.part_sums + ((int64_t)vec * 2 * L.ntiles + 2 * (int64_t)tile) * 2;
    if (threadIdx.x == 0) {
        ts[0] = l1;
        ts[1] = l2;
    }
    if (fb == lb) {
        const int64_t bs = L.offs[fb], be = L.offs[fb + 1];
        if (threadIdx.x == 0) {
            if (bs >= tile_start && be <= tile_start + TILE) {
                ratio_min(phi_bits, l1, l2, be - bs);
            } else {
                ps[0] = l1;         // first (and only) segment of the tile: slot 0
                ps[1] = l2;
            }
        }
        return;
    }
    // several blocks meet in this tile: segmented sums through LDS; the smallest ratio of the
    // segments that close here is collected in LDS first, one global atomic per tile
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) *reinterpret_cast<float4 *>(&S.val[local_base(k)]) = a[k];
    if (threadIdx.x == 0) {
        S.n_long = 0;
        tile_min = (unsigned long long)__double_as_longlong(1.0);
    }
    __syncthreads();
    const int nseg = lb - fb + 1;
    const bool head_open = L.offs[fb] < tile_start;
    const bool tail_open = L.offs[lb + 1] > tile_start + TILE;
    for (int sg = threadIdx.x; sg < nseg; sg += THREADS) {
        const int64_t b = fb + sg;
        const int64_t bs = L.offs[b], be = L.offs[b + 1];
        const int lo = (int)max(bs - tile_start, (int64_t)0);
        const int hi = (int)min(be - tile_start, (int64_t)n_valid);
        if (hi - lo > SMALL_SEG) {
            S.long_list[atomicAdd(&S.n_long, 1)] = sg;
            continue;
        }
        double s1 = 0.0, s2 = 0.0;
        for (int j = lo; j < hi; ++j) {
            const double x = S.val[j];
            s1 += x;
            s2 += x * x;
        }
        const bool open = (sg == 0 && head_open) || (sg == nseg - 1 && tail_open);
        if (open) {
            seg_sum[sg == 0 ? 0 : 1][0] = s1;
            seg_sum[sg == 0 ? 0 : 1][1] = s2;
        } else {
            ratio_min(&tile_min, s1, s2, be - bs);
        }
    }
    __syncthreads();
    const int n_long = S.n_long;
    for (int q = wave_id(); q < n_long; q += NWAVES) {
        const int sg = S.long_list[q];
        const int64_t b = fb + sg;
        const int64_t bs = L.offs[b], be = L.offs[b + 1];
        const int lo = (int)max(bs - tile_start, (int64_t)0);
        const int hi = (int)min(be - tile_start, (int64_t)n_valid);
        double s1 = 0.0, s2 = 0.0;
        for (int j = lo + lane_id(); j < hi; j += 64) {
            const double x = S.val[j];
            s1 += x;
            s2 += x * x;
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        const bool open = (sg == 0 && head_open) || (sg == nseg - 1 && tail_open);
        if (lane_id() == 0) {
            if (open) {
                seg_sum[sg == 0 ? 0 : 1][0] = s1;
                seg_sum[sg == 0 ? 0 : 1][1] = s2;
            } else {
                ratio_min(&tile_min, s1, s2, be - bs);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (tile_min != (unsigned long long)__double_as_longlong(1.0)) atomicMin(phi_bits, tile_min);
        if (head_open) {
            ps[0] = seg_sum[0][0];
            ps[1] = seg_sum[0][1];
        }
        if (tail_open) {
            ps[2] = seg_sum[1][0];
            ps[3] = seg_sum[1][1];
        }
    }
    __syncthreads();            // S.val and seg_sum are free again
}

__global__ __launch_bounds__(THREADS) void k_quality_tiles(Layout L, QualityArgs Q)
{
    __shared__ TileShared S;
    const int32_t tile = blockIdx.x;
    const int vec = blockIdx.y;
    const int n_valid = tile_valid(L, tile);
    float4 a[SUBROWS];
    load_tile(Q.v + (int64_t)vec * Q.stride + (int64_t)tile * TILE, a, n_valid);
    clear_past_end(a, n_valid);
    quality_of_tile(a, L, Q, tile, vec, n_valid, S);
}

// Sums of the n pairs at(0), at(1), ...: thread t adds t, t + THREADS, ... ascending, sixteen of them in flight (6240 tiles
// one after the other were 8 of this kernel's 10 us).
template <class At>
__device__ __forceinline__ void sum_pairs(int64_t n, At at, double &s1, double &s2)
{
    constexpr int DEEP = 16;
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += DEEP * THREADS) {
        double2 v[DEEP];
#pragma unroll
        for (int q = 0; q < DEEP; ++q) v[q] = *reinterpret_cast<const double2 *>(at(min(i0 + q * THREADS, n - 1)));
#pragma unroll
        for (int q = 0; q < DEEP; ++q) {
            const bool in = i0 + q * THREADS < n;           // the sums are of non-negative numbers: +0 changes nothing
            s1 += in ? v[q].x : 0.0;
            s2 += in ? v[q].y : 0.0;
        }
    }
}

// Workgroups 0 .. n_cross-1: one block that spans several tiles each.  The last
// workgroup of each vector: delta from the tile sums.
__global__ __launch_bounds__(THREADS) void k_quality_blocks(Layout L, QualityArgs Q, const int32_t *cross_blocks,
                                                            int n_cross)
{
    __shared__ double red[NWAVES];
    const int vec = blockIdx.y;
    double s1 = 0.0, s2 = 0.0;
    if ((int)blockIdx.x < n_cross) {
        const int64_t b = cross_blocks[blockIdx.x];
        const BlockSpan sp = block_span(L, b);
        const double *ps = Q.part_sums + (int64_t)vec * 2 * L.ntiles * 2;
        sum_pairs(sp.n, [&](int64_t i) { return ps + 2 * part_index(sp.t0 + i, sp); }, s1, s2);
        s1 = block_sum(s1, red);
        s2 = block_sum(s2, red);
        if (threadIdx.x == 0) ratio_min(Q.phi + vec, s1, s2, sp.be - sp.bs);
    } else {
        const double *ts = Q.tile_sums + (int64_t)vec * L.ntiles * 2;
        sum_pairs(L.ntiles, [&](int64_t i) { return ts + 2 * i; }, s1, s2);
        s1 = block_sum(s1, red);
        s2 = block_sum(s2, red);
        if (threadIdx.x == 0) Q.out[2 * (int64_t)vec + 1] = s2 > 0.0 ? s1 * s1 / ((double)L.d * s2) : 1.0;
    }
    if (threadIdx.x != 0) return;
    __builtin_amdgcn_s_waitcnt(0);      // the minimum has been taken
    if (atomicAdd(Q.done + vec, 1u) != (unsigned)n_cross) return;
    const unsigned long long phi = __hip_atomic_load(Q.phi + vec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Q.out[2 * (int64_t)vec] = __longlong_as_double((long long)phi);
    __hip_atomic_store(Q.phi + vec, (unsigned long long)__double_as_longlong(1.0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(Q.done + vec, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace ef
