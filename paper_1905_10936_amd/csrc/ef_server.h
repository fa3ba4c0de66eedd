// Server kernels of libef (Algorithm 4 of arxiv 1905.10936): see ef_tile.h for the tile scheme.
#pragma once
#include "ef_tile.h"
#include "ef_worker.h"

namespace ef {

// -------------------------------------------------------- server kernels ---

// (1/M) * acc as Algorithm 4 writes it: one correctly rounded fp32 division, or,
// when M is a power of two, the product with the exact reciprocal, which is the
// same real number and therefore rounds to the same bits.
__device__ __forceinline__ float mean_of(float acc, float Mf, float Minv)
{
    return Minv != 0.0f ? acc * Minv : acc / Mf;
}

constexpr int SERVER_CHUNK = 8;     // workers whose sign words are in flight together
constexpr int SCALE_GROUP = 4;      // dense tiles: workers whose scales are staged in LDS together ...
constexpr int SCALE_STAGE = TILE / 2;   // ... in this many floats

typedef unsigned vu4 __attribute__((ext_vector_type(4)));

// Bit matrix transpose: h[u] holds worker u's sign bits of 16 consecutive elements (bit e: element
// e); byte e of the result (element 0 in the lowest byte of .x) holds element e's bits of the eight
// workers (bit u: worker u).  The bytes are gathered into two 8x8 bit matrices, each transposed by
// swapping 1x1, 2x2 and 4x4 blocks across the diagonal.
__device__ __forceinline__ vu4 transpose_signs(const unsigned (&h)[SERVER_CHUNK])
{
    unsigned lo[2], hi[2];          // [half]: rows 0-3 and rows 4-7 of the matrix of elements 8*half .. 8*half+7
    {
        // v_perm_b32: selector values 0-3 take bytes of the second operand, 4-7 of the first
        const unsigned a = __builtin_amdgcn_perm(h[1], h[0], 0x05010400u), b = __builtin_amdgcn_perm(h[3], h[2], 0x05010400u);
        const unsigned c = __builtin_amdgcn_perm(h[5], h[4], 0x05010400u), d = __builtin_amdgcn_perm(h[7], h[6], 0x05010400u);
        lo[0] = __builtin_amdgcn_perm(b, a, 0x05040100u);
        lo[1] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        hi[0] = __builtin_amdgcn_perm(d, c, 0x05040100u);
        hi[1] = __builtin_amdgcn_perm(d, c, 0x07060302u);
    }
    unsigned out[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        unsigned x = lo[q], y = hi[q], t;
        t = (x ^ (x >> 7)) & 0x00AA00AAu;
        x ^= t ^ (t << 7);
        t = (y ^ (y >> 7)) & 0x00AA00AAu;
        y ^= t ^ (t << 7);
        t = (x ^ (x >> 14)) & 0x0000CCCCu;
        x ^= t ^ (t << 14);
        t = (y ^ (y >> 14)) & 0x0000CCCCu;
        y ^= t ^ (t << 14);
        out[2 * q] = (x & 0x0F0F0F0Fu) | ((y & 0x0F0F0F0Fu) << 4);
        out[2 * q + 1] = ((x >> 4) & 0x0F0F0F0Fu) | (y & 0xF0F0F0F0u);
    }
    return vu4{out[0], out[1], out[2], out[3]};
}

// LDS of server_values_whole.
constexpr int SUM_TABLE = 256;                          // floats: one sum per pattern of eight signs
constexpr int EXCHANGE_AT = SUM_TABLE;                  // 1 KiB per wavefront
constexpr int NIBBLE_AT = EXCHANGE_AT + NWAVES * 256;   // SERVER_CHUNK x 16 float4
constexpr int SERVER_LDS = NIBBLE_AT + SERVER_CHUNK * 64;      // floats

// p~ of a tile that lies inside one block b (Algorithm 4, server: decode and add the M payloads
// in worker order, divide by M, add the rescaled server residual tv).  Inside a block every element's
// sum over the first eight workers is one of 256 values, so the workgroup forms those 256 sums
// once, thread t the one of sign pattern t (in worker order from +0, divided by M if that is all of
// them: the operations Algorithm 4 writes, hence the same bits), and an element costs one LDS read.
// The pattern of an element is a byte: a lane loads each worker's bits of 16 consecutive elements,
// transposes the 8 x 16 bit matrix in registers and passes the bytes through LDS to the lanes that hold
// the elements (inside the wavefront).  Per 16 elements about 90 vector instructions, whatever M <= 8,
// where decoding worker by worker took 6 per four elements and worker and a division per element
// (2^28 elements in blocks of 2^20, same occupancy: M = 8 515 -> 491 us, M = 7 510 -> 478).
// Workers beyond the eighth are added one by one, eight at a time: entry (u, nibble) of a second table
// holds the four values +-s_u that a nibble of worker u's bits stands for, so four addends cost
// one bit-field extract and one 128-bit LDS read.
// Called by every thread of the workgroup; lds (SERVER_LDS floats) is free again on return.
template <bool MANY>
__device__ __forceinline__ void server_values_whole(const ServerArgs &A, int64_t tile_start, int32_t b,
                                                    const float4 (&tv)[SUBROWS], float4 (&p)[SUBROWS], float *lds)
{
    float acc[SUBROWS][4];
    const uint16_t *s16 = reinterpret_cast<const uint16_t *>(A.signs_in);
    const int64_t in_half = 4 * A.in_signs_stride;
    const int64_t half0 = (tile_start >> 4) + threadIdx.x;      // this lane's 16 elements: 16 * threadIdx.x of the tile
    const float r = A.r, Mf = A.Mf, Minv = A.Minv;
    unsigned *exchange = reinterpret_cast<unsigned *>(lds) + EXCHANGE_AT + wave_id() * 256;
    {
        unsigned h[SERVER_CHUNK];
        float sc[SERVER_CHUNK];
#pragma unroll
        for (int u = 0; u < SERVER_CHUNK; ++u) {
            const int i = min(u, A.M - 1);               // past M: a valid address whose value is not used
            h[u] = s16[(int64_t)i * in_half + half0];
            sc[u] = A.scales_in[(int64_t)i * A.in_scales_stride + b];
        }
        float sum = 0.0f;
#pragma unroll
        for (int u = 0; u < SERVER_CHUNK; ++u)
            if (u < A.M) sum = sum + signed_scale(sc[u], (threadIdx.x >> u) & 1u);
        lds[threadIdx.x] = MANY ? sum : mean_of(sum, Mf, Minv);
        *reinterpret_cast<vu4 *>(exchange + 4 * lane_id()) = transpose_signs(h);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) {
            const unsigned pat = exchange[64 * k + lane_id()];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] = lds[(pat >> (8 * c)) & 255u];
        }
    }
    if constexpr (MANY) {
        float4 *table = reinterpret_cast<float4 *>(lds + NIBBLE_AT);
        const unsigned sh = (unsigned)(lane_id() & 3) * 4u;
        for (int i0 = SERVER_CHUNK; i0 < A.M; i0 += SERVER_CHUNK) {
            unsigned h[SERVER_CHUNK];
            float sc[SERVER_CHUNK];
#pragma unroll
            for (int u = 0; u < SERVER_CHUNK; ++u) {
                const int i = min(i0 + u, A.M - 1);
                h[u] = s16[(int64_t)i * in_half + half0];
                sc[u] = A.scales_in[(int64_t)i * A.in_scales_stride + b];
            }
            if (i0 > SERVER_CHUNK) __syncthreads();      // the table is read no more
            if (threadIdx.x < SERVER_CHUNK * 16) {
                const int u = threadIdx.x >> 4, nib = threadIdx.x & 15;
                float su = sc[0];
#pragma unroll
                for (int q = 1; q < SERVER_CHUNK; ++q) su = (u == q) ? sc[q] : su;
                table[threadIdx.x] = make_float4(signed_scale(su, nib & 1), signed_scale(su, nib & 2),
                                                 signed_scale(su, nib & 4), signed_scale(su, nib & 8));
            }
            *reinterpret_cast<vu4 *>(exchange + 4 * lane_id()) =
                vu4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
            __syncthreads();
#pragma unroll
            for (int k = 0; k < SUBROWS; ++k) {
                // elements 256k + 4*lane .. +3 of the wavefront: half-word 16k + lane/4, nibble lane%4
                const vu4 w = *reinterpret_cast<const vu4 *>(exchange + 4 * (16 * k + (lane_id() >> 2)));
#pragma unroll
                for (int u = 0; u < SERVER_CHUNK; ++u) {
                    if (i0 + u < A.M) {
                        const unsigned two = w[u >> 1];
                        const float4 dv = table[u * 16 + ((two >> (sh + 16 * (u & 1))) & 15u)];
                        acc[k][0] = acc[k][0] + dv.x;
                        acc[k][1] = acc[k][1] + dv.y;
                        acc[k][2] = acc[k][2] + dv.z;
                        acc[k][3] = acc[k][3] + dv.w;
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] = mean_of(acc[k][c], Mf, Minv);
    }
    __syncthreads();            // lds is free again
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        p[k].x = acc[k][0] + r * tv[k].x;
        p[k].y = acc[k][1] + r * tv[k].y;
        p[k].z = acc[k][2] + r * tv[k].z;
        p[k].w = acc[k][3] + r * tv[k].w;
    }
}

// The same for a tile where several blocks meet (or the ragged end of the vector): a
// per-element segment index in LDS selects each worker's scale.  te: the tile of the server residual.
__device__ __forceinline__ void server_values_mixed(const Layout &L, const ServerArgs &A, int32_t tile, const TileRec &T, int n_valid,
                                                    const float *te, float4 (&p)[SUBROWS], TileShared &S)
{
    const int64_t tile_start = (int64_t)tile * TILE;
    const int32_t fb = T.fb, nseg = abs(T.nseg);
    float acc[SUBROWS][4];
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[k][c] = 0.0f;

    // this lane's 4 sign bits of sub-row k live in the 32-bit half-word hw0 + 8k
    const uint32_t *s32 = reinterpret_cast<const uint32_t *>(A.signs_in);
    const int64_t hw0 = (tile_start + local_base(0)) >> 5;
    const unsigned sh = (unsigned)(lane_id() & 7) * 4u;
    const int64_t n_hw = 2 * L.W;
    const int64_t in_hw = 2 * A.in_signs_stride;

    build_segment_index(L, tile, n_valid, fb, nseg, S);
    const ushort4 *seg4 = reinterpret_cast<const ushort4 *>(S.val);
    // The scales of the tile's segments are staged in LDS, SCALE_GROUP workers at a time where
    // they fit (one coalesced read per worker instead of a gather per element), and looked up
    // there; a tile with more segments than the stage holds gathers them from global memory.
    float *seg_scale = S.val + TILE / 2;            // the index takes the first half
    const int group = nseg * SCALE_GROUP <= SCALE_STAGE ? SCALE_GROUP : nseg <= SCALE_STAGE ? 1 : 0;
    if (group) {
        for (int i0 = 0; i0 < A.M; i0 += group) {
            uint32_t word[SCALE_GROUP][SUBROWS];
#pragma unroll
            for (int u = 0; u < SCALE_GROUP; ++u) {
                const int i = min(i0 + u, A.M - 1);      // past the group or M: loaded, not used
#pragma unroll
                for (int k = 0; k < SUBROWS; ++k) {
                    const int64_t hw = hw0 + 8 * k;
                    word[u][k] = (hw < n_hw) ? s32[(int64_t)i * in_hw + hw] : 0u;
                }
            }
            if (i0 > 0) __syncthreads();                 // the stage is read no more
            for (int u = 0; u < group && i0 + u < A.M; ++u) {
                const float *sc_i = A.scales_in + (int64_t)(i0 + u) * A.in_scales_stride + fb;
                for (int j = threadIdx.x; j < nseg; j += THREADS) seg_scale[u * nseg + j] = sc_i[j];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < SCALE_GROUP; ++u) {
                if (u < group && i0 + u < A.M) {
                    const float *sc_u = seg_scale + u * nseg;
#pragma unroll
                    for (int k = 0; k < SUBROWS; ++k) {
                        const unsigned nibble = (word[u][k] >> sh) & 0xFu;
                        const ushort4 sg = seg4[local_base(k) >> 2];
                        acc[k][0] = acc[k][0] + signed_scale(sc_u[sg.x], nibble & 1u);
                        acc[k][1] = acc[k][1] + signed_scale(sc_u[sg.y], nibble & 2u);
                        acc[k][2] = acc[k][2] + signed_scale(sc_u[sg.z], nibble & 4u);
                        acc[k][3] = acc[k][3] + signed_scale(sc_u[sg.w], nibble & 8u);
                    }
                }
            }
        }
    } else {
        for (int i = 0; i < A.M; ++i) {
            const float *sc_i = A.scales_in + (int64_t)i * A.in_scales_stride + fb;
#pragma unroll
            for (int k = 0; k < SUBROWS; ++k) {
                const int64_t hw = hw0 + 8 * k;
                const uint32_t word = (hw < n_hw) ? s32[(int64_t)i * in_hw + hw] : 0u;
                const unsigned nibble = (word >> sh) & 0xFu;
                const ushort4 sg = seg4[local_base(k) >> 2];
                acc[k][0] = acc[k][0] + signed_scale(sc_i[sg.x], nibble & 1u);
                acc[k][1] = acc[k][1] + signed_scale(sc_i[sg.y], nibble & 2u);
                acc[k][2] = acc[k][2] + signed_scale(sc_i[sg.z], nibble & 4u);
                acc[k][3] = acc[k][3] + signed_scale(sc_i[sg.w], nibble & 8u);
            }
        }
    }
    __syncthreads();            // S.val is free again
    float4 tv[SUBROWS];
    load_tile(te, tv, n_valid);
    const float r = A.r, Mf = A.Mf, Minv = A.Minv;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        p[k].x = mean_of(acc[k][0], Mf, Minv) + r * tv[k].x;
        p[k].y = mean_of(acc[k][1], Mf, Minv) + r * tv[k].y;
        p[k].z = mean_of(acc[k][2], Mf, Minv) + r * tv[k].z;
        p[k].w = mean_of(acc[k][3], Mf, Minv) + r * tv[k].w;
    }
}

// Layouts of dense tiles alone (25 M elements in blocks of 33, 7 workers: 86 us; blocks of 256, 4 workers, 16 M
// elements: 49.5, against 52.2 in a kernel with the whole tiles' code).  The residual tile is loaded after the
// payloads have been added up, which keeps the registers down.
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(7, 8)))
void k_server_mixed(Layout L, ScratchRef R, ServerArgs A, int set)
{
    const Scratch X = open_call(R);
    __shared__ TileShared S;
    const TileRec T = L.mixed_recs[blockIdx.x];
    const int32_t tile = T.tile;
    const int n_valid = tile_valid(L, tile);
    float *te = A.err + (int64_t)tile * TILE;
    float4 p[SUBROWS];
    server_values_mixed(L, A, tile, T, n_valid, te, p, S);
    compress_mixed(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S);
    snapshot_call(R);           // there may be no whole tiles
}

// p~ of a tile of a few segments (see compress_few): as server_values_whole, with a table of sums for one segment
// after the other and every thread's elements masked by the segment's range.
template <bool MANY>
__device__ __forceinline__ void server_values_few(const Layout &L, const ServerArgs &A, const TileRec &T, int64_t tile_start,
                                                  const float *te, int n_valid, float4 (&p)[SUBROWS], float *lds, const int *bound)
{
    float acc[SUBROWS][4];
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[k][c] = 0.0f;
    const uint16_t *s16 = reinterpret_cast<const uint16_t *>(A.signs_in);
    const int64_t in_half = 4 * A.in_signs_stride, half0 = (tile_start >> 4) + threadIdx.x;
    const bool in = half0 < 4 * L.W;                     // the ragged end
    const float r = A.r, Mf = A.Mf, Minv = A.Minv;
    unsigned *exchange = reinterpret_cast<unsigned *>(lds) + EXCHANGE_AT + wave_id() * 256;
    float4 *nibbles = reinterpret_cast<float4 *>(lds + NIBBLE_AT);
#pragma unroll 1
    for (int i0 = 0; i0 < (MANY ? A.M : 1); i0 += SERVER_CHUNK) {
        const int mine = min(i0 + (lane_id() & (SERVER_CHUNK - 1)), A.M - 1);
        const float *sc_i = A.scales_in + (int64_t)mine * A.in_scales_stride + T.fb;
        float sc = sc_i[0];                              // lane u: the segment's scale from worker i0 + u
        {
            unsigned h[SERVER_CHUNK];
#pragma unroll
            for (int u = 0; u < SERVER_CHUNK; ++u)
                h[u] = in ? s16[(int64_t)min(i0 + u, A.M - 1) * in_half + half0] : 0u;
            const vu4 row = !MANY || i0 == 0 ? transpose_signs(h)
                                    : vu4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
            *reinterpret_cast<vu4 *>(exchange + 4 * lane_id()) = row;
        }
        __syncthreads();                                 // (the first time: the bounds are there)
#pragma unroll 1
        for (int sg = 0; sg < T.nseg; ++sg) {
            const int lo = few_bound(bound, sg), hi = few_bound(bound, sg + 1);
            const unsigned n = (unsigned)(hi - lo);
            const float now = sc;
            if (sg + 1 < T.nseg) sc = sc_i[sg + 1];
            if (!MANY || i0 == 0) {
                float sum = 0.0f;
#pragma unroll
                for (int u = 0; u < SERVER_CHUNK; ++u) {
                    const float s = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(now), u));
                    if (u < A.M) sum = sum + signed_scale(s, (threadIdx.x >> u) & 1u);
                }
                lds[threadIdx.x] = MANY ? sum : mean_of(sum, Mf, Minv);
                __syncthreads();
#pragma unroll
                for (int k = 0; k < SUBROWS; ++k) {
                    if (!few_touches(k, lo, hi)) continue;
                    const unsigned pat = exchange[64 * k + lane_id()];
                    const int j = local_base(k) - lo;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float v = lds[(pat >> (8 * c)) & 255u];
                        acc[k][c] = (unsigned)(j + c) < n ? v : acc[k][c];
                    }
                }
            } else {
                const float su = __shfl(now, (int)(threadIdx.x >> 4) & (SERVER_CHUNK - 1));
                if (threadIdx.x < SERVER_CHUNK * 16) {
                    const unsigned nib = threadIdx.x & 15u;
                    nibbles[threadIdx.x] = make_float4(signed_scale(su, nib & 1u), signed_scale(su, nib & 2u),
                                                       signed_scale(su, nib & 4u), signed_scale(su, nib & 8u));
                }
                __syncthreads();
                const unsigned sh = (unsigned)(lane_id() & 3) * 4u;
#pragma unroll
                for (int k = 0; k < SUBROWS; ++k) {
                    if (!few_touches(k, lo, hi)) continue;
                    const vu4 w = *reinterpret_cast<const vu4 *>(exchange + 4 * (16 * k + (lane_id() >> 2)));
                    const int j = local_base(k) - lo;
#pragma unroll
                    for (int u = 0; u < SERVER_CHUNK; ++u) {
                        if (i0 + u < A.M) {
                            const float4 dv = nibbles[u * 16 + ((w[u >> 1] >> (sh + 16 * (u & 1))) & 15u)];
                            acc[k][0] = (unsigned)(j + 0) < n ? acc[k][0] + dv.x : acc[k][0];
                            acc[k][1] = (unsigned)(j + 1) < n ? acc[k][1] + dv.y : acc[k][1];
                            acc[k][2] = (unsigned)(j + 2) < n ? acc[k][2] + dv.z : acc[k][2];
                            acc[k][3] = (unsigned)(j + 3) < n ? acc[k][3] + dv.w : acc[k][3];
                        }
                    }
                }
            }
            __syncthreads();                             // the table, and after the last segment the exchange, are free
        }
    }
    if (MANY) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] = mean_of(acc[k][c], Mf, Minv);
    }
    float4 tv[SUBROWS];             // loaded only now: few registers
    load_tile(te, tv, n_valid);
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        p[k].x = acc[k][0] + r * tv[k].x;
        p[k].y = acc[k][1] + r * tv[k].y;
        p[k].z = acc[k][2] + r * tv[k].z;
        p[k].w = acc[k][3] + r * tv[k].w;
    }
}

// Server part of Algorithm 4, all tiles in one launch, one workgroup per tile, in the order of k_worker_tiles.  p~ as
// above, then compressed like a worker's p; the workgroup of a whole tile waits in the kernel for its block's scale.
// Bound by HBM and, where blocks wait for their scale, by the workgroups resident meanwhile.  Workgroups per CU:
//   whole tiles only    eight (64 VGPRs; 2^28 elements, 8 workers, blocks of 2^20: 457 us against 465 at seven, 491 at six)
//   tiles of few segments, or MANY    seven (68 VGPRs, none spilled; with the dense tiles' code at eight 39 are)
//   dense tiles         six (80 VGPRs; 643 965 tiny blocks, 2 workers: 46.3 us against 49.4 at seven, where 6 spill;
//                       16 workers, 300 000: 51.0 against 52.8)
// MANY: more than SERVER_CHUNK workers.
template <bool SEGMENTS>
struct ServerShared : SyncShared {
    float val[SERVER_LDS];
};
template <>
struct ServerShared<true> : TileShared {};
static_assert(SERVER_LDS <= TILE, "one array for the sum tables and for the segments");

template <int TILES, bool MANY>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(TILES == DENSE_TILES ? 6 : TILES == FEW_TILES || MANY ? 7 : 8, 8)))
void k_server_tiles(Layout L, ScratchRef R, ServerArgs A, int set)
{
    constexpr bool MIXED = TILES != ALL_WHOLE;
    __shared__ __align__(16) ServerShared<MIXED> S;
    float *lds = S.val;
    float4 tv[SUBROWS], p[SUBROWS];
    if (!MIXED) {
        // tile i is workgroup i's: its residual is asked for before anything is looked up
        load_tile(A.err + (int64_t)blockIdx.x * TILE, tv, TILE);
        __builtin_amdgcn_sched_barrier(0);
    }
    const Scratch X = open_call(R);
    const TileRec T = MIXED ? L.grid_tiles[blockIdx.x] : L.tiles[blockIdx.x];
    const int32_t tile = MIXED ? T.tile : (int32_t)blockIdx.x;
    const int64_t tile_start = (int64_t)tile * TILE;
    const int n_valid = MIXED ? tile_valid(L, tile) : TILE;
    float *te = A.err + tile_start;
    if (!MIXED || T.words < 0) {
        if (MIXED) load_tile(te, tv, TILE);
        Posted P;
        const BlockSpan sp = span_of(T.bs(), T.be());
        const LoadedCorrection corr = loaded_correction(L, T.fb, X, set);
        correct_loaded_residual(tv, corr);
        server_values_whole<MANY>(A, tile_start, T.fb, tv, p, lds);
        const int kind = compress_uniform(p, L, tile, T.fb, sp, TILE, A.signs, A.scales, te, X, set, S, P);
        resolve_posted(P, L, X, set, A.scales, S);
        if (kind == UNI_PENDING) finish_uniform(p, tile, TILE, sp, 0ull, te, L, X, set, S);
    } else if constexpr (MIXED) {
        if (TILES == DENSE_TILES && T.nseg < 0) {
            server_values_mixed(L, A, tile, T, n_valid, te, p, S);
            compress_mixed(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S);
            snapshot_call(R);
            return;
        }
        __shared__ FewShared F;
        few_bounds(L, T, tile_start, n_valid, F.bound);
        server_values_few<MANY>(L, A, T, tile_start, te, n_valid, p, lds, F.bound);
        compress_few(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S, F, lds);
    }
    snapshot_call(R);
}

}  // namespace ef
