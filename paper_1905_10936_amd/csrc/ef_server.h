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

// The same for a thread's elements, with one branch.
__device__ __forceinline__ void mean_of_all(float (&acc)[SUBROWS][4], float Mf, float Minv)
{
    if (Minv != 0.0f) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] *= Minv;
    } else {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] /= Mf;
    }
}

constexpr int SERVER_CHUNK = 8;     // workers whose sign words are in flight together
constexpr int SCALE_GROUP = 4;      // dense tiles: workers whose scales are staged in LDS together ...
constexpr int SCALE_STAGE = TILE / 2;   // ... in this many floats

typedef unsigned vu4 __attribute__((ext_vector_type(4)));

// Bit matrix transpose: h[u] holds worker u's sign bits of 16 consecutive elements (bit e: element
// e); byte e of the result (element 0 in the lowest byte of .x) holds element e's bits of the eight
// workers (bit u: worker u).  Each step exchanges one bit of u, first a register number, with one bit of e, first
// a bit position; the last puts an element's byte where it belongs (40 instructions).
__device__ __forceinline__ vu4 transpose_signs(const unsigned (&h)[SERVER_CHUNK])
{
    unsigned q[4];                  // bit 0 of u <-> bit 0 of e; elements of odd e in the upper half
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const unsigned a = h[2 * r], b = h[2 * r + 1];
        const unsigned even = (a & 0x5555u) | ((b << 1) & ~0x5555u), odd = ((a >> 1) & 0x5555u) | (b & ~0x5555u);
        // v_perm_b32: selector values 0-3 take bytes of the second operand, 4-7 of the first
        q[r] = __builtin_amdgcn_perm(odd, even, 0x05040100u);
    }
#pragma unroll
    for (int r = 0; r < 4; r += 2) {        // bit 1 <-> bit 1
        const unsigned a = q[r], b = q[r + 1];
        q[r] = (a & 0x33333333u) | ((b << 2) & ~0x33333333u);
        q[r + 1] = ((a >> 2) & 0x33333333u) | (b & ~0x33333333u);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {           // bit 2 <-> bit 2
        const unsigned a = q[r], b = q[r + 2];
        q[r] = (a & 0x0F0F0F0Fu) | ((b << 4) & ~0x0F0F0F0Fu);
        q[r + 2] = ((a >> 4) & 0x0F0F0F0Fu) | (b & ~0x0F0F0F0Fu);
    }
    // element e is byte 2 * (bit 0 of e) + (bit 3 of e) of q[bits 1 and 2 of e]
    return vu4{__builtin_amdgcn_perm(q[1], q[0], 0x06040200u), __builtin_amdgcn_perm(q[3], q[2], 0x06040200u),
               __builtin_amdgcn_perm(q[1], q[0], 0x07050301u), __builtin_amdgcn_perm(q[3], q[2], 0x07050301u)};
}

// s if bit u of minus is 0, else -s
__device__ __forceinline__ float negated_by(float s, unsigned minus, int u)
{
    return __uint_as_float(__float_as_uint(s) ^ ((minus << (31 - u)) & 0x80000000u));
}

// This lane's sign bits of workers i0 .. i0 + 7 (past M: the last worker's again, not used): 16 consecutive elements,
// 16 * threadIdx.x of the tile.  Asked for ahead of everything that is looked up by block.
__device__ __forceinline__ void load_sign_halves(const ServerArgs &A, int64_t tile_start, int i0, unsigned (&h)[SERVER_CHUNK])
{
    const uint16_t *row = reinterpret_cast<const uint16_t *>(A.signs_in + (int64_t)i0 * A.in_signs_stride) + (tile_start >> 4);
#pragma unroll
    for (int u = 0; u < SERVER_CHUNK; ++u) {
        h[u] = row[threadIdx.x];
        row += i0 + u + 1 < A.M ? 4 * A.in_signs_stride : 0;
    }
}
// Block b's scales from workers i0 .. i0 + 7; past M 0, which changes no sum.
__device__ __forceinline__ void load_scales(const ServerArgs &A, int32_t b, int i0, float (&sc)[SERVER_CHUNK])
{
    const float *at = A.scales_in + (int64_t)i0 * A.in_scales_stride + b;
#pragma unroll
    for (int u = 0; u < SERVER_CHUNK; ++u) {
        const float s = *at;
        sc[u] = i0 + u < A.M ? s : 0.0f;
        at += i0 + u + 1 < A.M ? A.in_scales_stride : 0;
    }
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
// h: the sign bits of the ninth to the sixteenth, asked for with those of the first eight, as are the scales of the table's
// makers.  (12 000 tiles in blocks of 64: 16 workers 98.5 -> 93.1 us, 11 workers 98.0 -> 93.2.)
// Called by every thread of the workgroup; lds (SERVER_LDS floats) is free again on return.
__device__ __forceinline__ float nibble_scale(const ServerArgs &A, int32_t b, int i0)
{
    return A.scales_in[(int64_t)min(i0 + (int)(threadIdx.x >> 4), A.M - 1) * A.in_scales_stride + b];
}
template <bool MANY>
__device__ __forceinline__ void server_values_whole(const ServerArgs &A, int64_t tile_start, int32_t b, const unsigned (&h0)[SERVER_CHUNK],
                                                    unsigned (&h)[SERVER_CHUNK], const float4 (&tv)[SUBROWS], float4 (&p)[SUBROWS], float *lds)
{
    // the scale of the worker whose nibbles this thread tabulates, asked for ahead of the tile's values
    float next = 0.0f;
    if (MANY && threadIdx.x < SERVER_CHUNK * 16) next = nibble_scale(A, b, SERVER_CHUNK);
    float acc[SUBROWS][4];
    const float r = A.r, Mf = A.Mf, Minv = A.Minv;
    unsigned *exchange = reinterpret_cast<unsigned *>(lds) + EXCHANGE_AT + wave_id() * 256;
    {
        float sc[SERVER_CHUNK];
        load_scales(A, b, 0, sc);
        float sum = 0.0f;
        const unsigned minus = ~threadIdx.x;
#pragma unroll
        for (int u = 0; u < SERVER_CHUNK; ++u) sum = sum + negated_by(sc[u], minus, u);
        lds[threadIdx.x] = MANY ? sum : mean_of(sum, Mf, Minv);
        *reinterpret_cast<vu4 *>(exchange + 4 * lane_id()) = transpose_signs(h0);
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
            if (i0 > SERVER_CHUNK) {
                load_sign_halves(A, tile_start, i0, h);
                __syncthreads();                         // the table is read no more
            }
            if (threadIdx.x < SERVER_CHUNK * 16) {
                const int nib = threadIdx.x & 15;
                const float su = i0 + (int)(threadIdx.x >> 4) < A.M ? next : 0.0f;
                if (i0 + SERVER_CHUNK < A.M) next = nibble_scale(A, b, i0 + SERVER_CHUNK);
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
                    // past M +-0, which changes no sum (one that began with +0 is never -0): no branch between the reads
                    const unsigned two = w[u >> 1];
                    const float4 dv = table[u * 16 + ((two >> (sh + 16 * (u & 1))) & 15u)];
                    acc[k][0] = acc[k][0] + dv.x;
                    acc[k][1] = acc[k][1] + dv.y;
                    acc[k][2] = acc[k][2] + dv.z;
                    acc[k][3] = acc[k][3] + dv.w;
                }
            }
        }
        mean_of_all(acc, Mf, Minv);
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
    const float r = A.r;
    mean_of_all(acc, A.Mf, A.Minv);
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        p[k].x = acc[k][0] + r * tv[k].x;
        p[k].y = acc[k][1] + r * tv[k].y;
        p[k].z = acc[k][2] + r * tv[k].z;
        p[k].w = acc[k][3] + r * tv[k].w;
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
    const unsigned left = compress_mixed(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S);
    end_call(left, R, X, S);    // there may be no whole tiles
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
    if (MANY) mean_of_all(acc, Mf, Minv);
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

// Two whole tiles of one block, next to each other, as one workgroup's work: wavefront w has the elements
// 2048w .. 2048w + 2047 of the pair as two quarters of a tile each laid out like a quarter elsewhere, so that a
// tile's sum is formed in the same order.  One offset, in the middle of a wavefront's 8 KiB, serves all of a thread's eight
// accesses, which lie within what an instruction can add to it (from its start on, the upper half needed four addresses).
__device__ __forceinline__ float *pair_part(float *te, int half, int k)
{
    unsigned middle = (2u * (threadIdx.x >> 6) + 1u) * 4096u + (threadIdx.x & 63u) * 16u;
    asm("" : "+v"(middle));             // one register, not an address and its upper half's
    return reinterpret_cast<float *>(reinterpret_cast<char *>(te) + middle) + (half - 1) * 1024 + k * 256;
}

// As transpose_signs, for 32 consecutive elements: dword j of the result holds the bytes of elements 4j .. 4j + 3.
__device__ __forceinline__ void transpose_signs32(const unsigned (&h)[SERVER_CHUNK], vu4 (&out)[2])
{
    unsigned q[SERVER_CHUNK];
#pragma unroll
    for (int u = 0; u < 8; u += 2) {            // bit 0 of u <-> bit 0 of e
        const unsigned a = h[u], b = h[u + 1];
        q[u] = (a & 0x55555555u) | ((b << 1) & ~0x55555555u);
        q[u + 1] = ((a >> 1) & 0x55555555u) | (b & ~0x55555555u);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {               // bit 1 <-> bit 1
        const int u = (i & 1) | ((i & 2) << 1);
        const unsigned a = q[u], b = q[u + 2];
        q[u] = (a & 0x33333333u) | ((b << 2) & ~0x33333333u);
        q[u + 2] = ((a >> 2) & 0x33333333u) | (b & ~0x33333333u);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {               // bit 2 <-> bit 2
        const unsigned a = q[u], b = q[u + 4];
        q[u] = (a & 0x0F0F0F0Fu) | ((b << 4) & ~0x0F0F0F0Fu);
        q[u + 4] = ((a >> 4) & 0x0F0F0F0Fu) | (b & ~0x0F0F0F0Fu);
    }
    // element e is byte (bits 3 and 4 of e) of q[bits 0 to 2 of e]: 4 x 4 bytes transposed, twice
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const unsigned a = q[4 * g], b = q[4 * g + 1], c = q[4 * g + 2], d = q[4 * g + 3];
        const unsigned ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
        const unsigned cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
        out[0][g] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
        out[0][g + 2] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
        out[1][g] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
        out[1][g + 2] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
    }
}

// LDS of server_pair (32-bit words): the wavefronts' exchanges (2 KiB each), and the table of sums, over the first eight workers or
// the first twelve; beyond those, the values four more workers' signs stand for.
constexpr int PAIR_WORKERS = 2 * SERVER_CHUNK;
constexpr int PAIR_EXCHANGE = NWAVES * 512;
constexpr int TWELVE = SERVER_CHUNK + 4;
constexpr int PAIR_SUMS = 1 << TWELVE;
constexpr int PAIR_VALUES = 16 * 4;

__device__ __forceinline__ void load_sign_dwords(const ServerArgs &A, int64_t start, int i0, unsigned (&h)[SERVER_CHUNK])
{
    const unsigned *row = reinterpret_cast<const unsigned *>(A.signs_in + (int64_t)i0 * A.in_signs_stride) + (start >> 5);
#pragma unroll
    for (int u = 0; u < SERVER_CHUNK; ++u) {
        h[u] = row[threadIdx.x];
        row += i0 + u + 1 < A.M ? 2 * A.in_signs_stride : 0;
    }
}

// A thread's bytes of a pair, by half and sub-row: dword (h, k) holds the bytes of elements 0 to 3 of pair_part(h, k).
__device__ __forceinline__ unsigned pair_bytes(const unsigned *exchange, int half, int k) { return exchange[256 * half + 64 * k + lane_id()]; }
__device__ __forceinline__ void put_pair_bytes(unsigned *exchange, const unsigned (&h)[SERVER_CHUNK])
{
    vu4 bytes[2];
    transpose_signs32(h, bytes);
    *reinterpret_cast<vu4 *>(exchange + 8 * lane_id()) = bytes[0];
    *reinterpret_cast<vu4 *>(exchange + 8 * lane_id() + 4) = bytes[1];
}
// Sum over the first eight workers of sign pattern threadIdx.x.
__device__ __forceinline__ float eight_sum(const ServerArgs &A, int32_t b)
{
    float sc[SERVER_CHUNK];
    load_scales(A, b, 0, sc);
    float sum = 0.0f;
    const unsigned minus = ~threadIdx.x;
#pragma unroll
    for (int u = 0; u < SERVER_CHUNK; ++u) sum = sum + negated_by(sc[u], minus, u);
    return sum;
}

// p~ of a pair of up to eight workers, as server_values_whole.  v: the server residual's tiles, then p~.  sums: SUM_TABLE floats.
__device__ __forceinline__ void server_values_pair(const ServerArgs &A, int32_t b, const unsigned (&h)[SERVER_CHUNK],
                                                   float4 (&v)[2][SUBROWS], unsigned *exchanges, float *sums)
{
    const float r = A.r;
    unsigned *exchange = exchanges + wave_id() * 512;
    sums[threadIdx.x] = mean_of(eight_sum(A, b), A.Mf, A.Minv);
    put_pair_bytes(exchange, h);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) {
            const unsigned pat = pair_bytes(exchange, q, k);
            v[q][k].x = sums[pat & 255u] + r * v[q][k].x;
            v[q][k].y = sums[(pat >> 8) & 255u] + r * v[q][k].y;
            v[q][k].z = sums[(pat >> 16) & 255u] + r * v[q][k].z;
            v[q][k].w = sums[pat >> 24] + r * v[q][k].w;
        }
}

// The same for nine to sixteen workers (PAIR_WORKERS).  The table has the sums over the first twelve, in worker order from +0, 4096
// of them: thread t makes the sixteen that begin with pattern t, 30 additions on top of the eight, where adding the four workers
// one by one takes each of its 32 elements four additions, four reads and as many bit fields.  The next four are added one by
// one; their values +-s come in one read for an element.  An element's sixteen bits are two bytes, transposed
// and exchanged one after the other.  Server call, 354 M of a transformer, us: 11 workers 845 -> 732, 14 900 -> 791, 16 870 -> 808;
// 25 M of a bottleneck network, 16 workers: 76 -> 70.
// sums: PAIR_SUMS floats; values: PAIR_VALUES.
__device__ __forceinline__ void server_values_pair_many(const ServerArgs &A, int32_t b, const unsigned (&h0)[SERVER_CHUNK],
                                                        const unsigned (&h1)[SERVER_CHUNK], float4 (&v)[2][SUBROWS],
                                                        unsigned *exchanges, float *sums, float *values)
{
    const float r = A.r, Mf = A.Mf, Minv = A.Minv;
    const bool more = A.M > TWELVE;
    unsigned *exchange = exchanges + wave_id() * 512;
    {
        // past M: +-0, which changes no sum (one that began with +0 is never -0)
        float sum[16], sc[4];
        sum[0] = eight_sum(A, b);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float s = A.scales_in[(int64_t)min(SERVER_CHUNK + u, A.M - 1) * A.in_scales_stride + b];
            sc[u] = SERVER_CHUNK + u < A.M ? s : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i = 0; i < (1 << u); ++i) {
                sum[i + (1 << u)] = sum[i] + sc[u];
                sum[i] = sum[i] + -sc[u];
            }
#pragma unroll
        for (int i = 0; i < 16; ++i) sums[256 * i + threadIdx.x] = more ? sum[i] : mean_of(sum[i], Mf, Minv);
    }
    if (more && threadIdx.x < PAIR_VALUES) {
        const int i = TWELVE + (int)(threadIdx.x & 3u);
        float s = A.scales_in[(int64_t)min(i, A.M - 1) * A.in_scales_stride + b];
        s = i < A.M ? s : 0.0f;
        values[threadIdx.x] = signed_scale(s, (threadIdx.x >> (2 + (threadIdx.x & 3u))) & 1u);
    }
    unsigned first[2][SUBROWS];
    put_pair_bytes(exchange, h0);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) first[q][k] = pair_bytes(exchange, q, k);
    put_pair_bytes(exchange, h1);
    __syncthreads();
    // four elements at a time: more in flight are more registers than there are
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) {
            const unsigned second = pair_bytes(exchange, q, k);
            // two elements' sixteen bits to a word
            const unsigned w[2] = {__builtin_amdgcn_perm(second, first[q][k], 0x05010400u), __builtin_amdgcn_perm(second, first[q][k], 0x07030602u)};
            float acc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = sums[(w[c >> 1] >> (16 * (c & 1))) & (unsigned)(PAIR_SUMS - 1)];
            if (more) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float4 dv = *reinterpret_cast<const float4 *>(values + 4 * ((w[c >> 1] >> (16 * (c & 1) + TWELVE)) & 15u));
                    acc[c] = (((acc[c] + dv.x) + dv.y) + dv.z) + dv.w;
                }
                if (Minv != 0.0f) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] *= Minv;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] /= Mf;
                }
            }
            v[q][k].x = acc[0] + r * v[q][k].x;
            v[q][k].y = acc[1] + r * v[q][k].y;
            v[q][k].z = acc[2] + r * v[q][k].z;
            v[q][k].w = acc[3] + r * v[q][k].w;
            // formed here: put off to where they are used, the 32 sums and the residuals need a register each
            asm volatile("" : "+v"(v[q][k].x), "+v"(v[q][k].y), "+v"(v[q][k].z), "+v"(v[q][k].w));
            __builtin_amdgcn_sched_barrier(0);
        }
}

// A pair from loads to stores (compress_uniform and settle_uniform for both tiles at once).  Returns arrived()'s answer.
template <bool MANY>
__device__ __forceinline__ unsigned server_pair(const Layout &L, const ServerArgs &A, const TileRec &T, const Scratch &X, int set,
                                                SyncShared &S, float *lds, float *more)
{
    const int64_t start = (int64_t)T.tile * TILE;
    float *te = A.err + start;
    unsigned h[SERVER_CHUNK], h1[SERVER_CHUNK];
    float4 v[2][SUBROWS];
    load_sign_dwords(A, start, 0, h);
    if (MANY) load_sign_dwords(A, start, SERVER_CHUNK, h1);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) v[q][k] = stream_load4(pair_part(te, q, k));
    __builtin_amdgcn_sched_barrier(0);
    const BlockSpan sp = span_of(T.bs(), T.be());
    const LoadedCorrection corr = loaded_correction(L, T.fb, X, set);
    correct_loaded_residual(v[0], corr);
    correct_loaded_residual(v[1], corr);
    if constexpr (MANY)
        server_values_pair_many(A, T.fb, h, h1, v, reinterpret_cast<unsigned *>(more), lds, more + PAIR_EXCHANGE);
    else
        server_values_pair(A, T.fb, h, v, reinterpret_cast<unsigned *>(lds), more);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        store_quarter_signs<false>(sign_half(v[q], TILE), A.signs, (start >> 6) + (2 * wave_id() + q) * 16, L.W);
        const double quarter = wave_sum(abs_sum(v[q], TILE));
        if (lane_id() == 0) S.red[2 * wave_id() + q] = quarter;
    }
    __syncthreads();
    const double first = ((S.red[0] + S.red[1]) + S.red[2]) + S.red[3], second = ((S.red[4] + S.red[5]) + S.red[6]) + S.red[7];
    __syncthreads();
    bool finished = false;
    float s = 0.f;
    if (threadIdx.x < 2) {
        const unsigned long long w = (unsigned long long)__double_as_longlong(threadIdx.x ? second : first);
        __hip_atomic_store(set_part(X, L, set) + 2 * ((int64_t)T.tile + threadIdx.x), w | (set_tag(X, set) ? TAG_BIT : 0ull),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const unsigned before = arrive(X, S);
    const bool counted = is_counted(L, sp), kept = counted || (L.keep > 0 && (int64_t)T.tile >= first_kept(L, sp));
    const bool forms = (counted || L.keep > 0) && (int64_t)T.tile + 1 == last_whole_tile(sp);
    if (kept || forms) finished = block_scale(forms, T.fb, sp, L, X, set, A.scales, S, 0, &s) && kept;    // else parked like the others of its block
    const unsigned left = arrived(before, X);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (finished)
#pragma unroll
            for (int k = 0; k < SUBROWS; ++k) residual4(v[q][k], s);
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) stream_store4(pair_part(te, q, k), v[q][k]);
    }
    if (kept && !finished) park_segment(T.tile, 0, true, X, set, S);
    return left;
}

// Server part of Algorithm 4, all tiles in one launch, in the order of k_worker_tiles.  p~ as
// above, then compressed like a worker's p; the workgroup of a whole tile waits in the kernel for its block's scale.
// Bound by HBM and, where blocks wait for their scale, by the tiles resident meanwhile: a workgroup's life is
// half decoding, half the wait for the slowest tile of its block.  PAIRS: two whole tiles of a block to a workgroup, both
// loaded ahead of all else, so that a CU has 14 tiles instead of 8 (12 instead of 7 beyond eight workers), one wait and
// one table for two.  7 workers, 25 M elements of a bottleneck network: 54.9 -> 44.3 us; 16 workers, 354 M of a
// transformer, whose blocks of 1025 tiles then finish in one pass: 1092 -> 907 (870 with first_kept and gather_scale as they are); 8 workers, 2^28 in blocks of 2^20:
// 450 -> 400.  Where nothing waits (every block beyond the limit) one tile to a workgroup is the faster (4
// workers, 2^26: 4 us less), and elsewhere by server_pairs (ef_layout.h).  Workgroups per CU:
//   pairs               seven (72 VGPRs), MANY six (77; 25 KB of LDS); one less: 46.3 us, MANY 916 against 826
//   whole tiles only    eight (64 VGPRs; 2^28 elements, 8 workers, blocks of 2^20: 457 us against 465 at seven, 491 at six)
//   tiles of few segments    eight (61 VGPRs), MANY seven (70); MANY on whole tiles only seven (68)
//   dense tiles         six (80 VGPRs; 643 965 tiny blocks, 2 workers: 46.3 us against 49.4 at seven, where 6 spill;
//                       16 workers, 300 000: 51.0 against 52.8)
// MANY: more than SERVER_CHUNK workers.
template <bool SEGMENTS, int FLOATS>
struct ServerShared : SyncShared {
    alignas(16) float val[FLOATS];      // read 128 bits at a time
};
template <int FLOATS>
struct ServerShared<true, FLOATS> : TileShared {
    static_assert(FLOATS <= TILE, "one array for the sum tables, the exchanges and the segments");
};

// Workgroups per CU.
constexpr int server_occupancy(int tiles, bool many, bool pairs)
{
    return pairs ? (many ? 6 : 7) : tiles == DENSE_TILES ? 6 : tiles == FEW_TILES || many ? 7 : 8;
}

// Pairs of more than eight workers leave the end of their calls to k_tail: the code for it costs the pairs more than that
// (354 M of a transformer, 14 workers: 730 us without, 783 with it).
// Nor do the kernels with dense tiles: blocks with whole tiles leave their segments in those to k_tail anyway, and the code costs
// them 5 % (a million tiny blocks and four of 8 Mi, 4 workers: 111 -> 117 us).
constexpr bool server_ends(int tiles, bool many, bool pairs) { return tiles != DENSE_TILES && !(many && pairs); }

template <int TILES, bool MANY, bool PAIRS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(server_occupancy(TILES, MANY, PAIRS), 8)))
void k_server_tiles(Layout L, ScratchRef R, ServerArgs A, int set)
{
    constexpr bool MIXED = TILES != ALL_WHOLE;
    constexpr int FOR_PAIRS = PAIRS ? (MANY ? PAIR_SUMS : PAIR_EXCHANGE) : 0;
    __shared__ __align__(16) ServerShared<MIXED, (FOR_PAIRS > SERVER_LDS ? FOR_PAIRS : SERVER_LDS)> S;
    float *lds = S.val;
    float4 tv[SUBROWS], p[SUBROWS];
    unsigned h[SERVER_CHUNK], h1[SERVER_CHUNK];
    if (!MIXED && !PAIRS) {
        // tile i is workgroup i's: its sign words and its residual are asked for before anything is looked up
        load_sign_halves(A, (int64_t)blockIdx.x * TILE, 0, h);
        if (MANY) load_sign_halves(A, (int64_t)blockIdx.x * TILE, SERVER_CHUNK, h1);
        load_tile(A.err + (int64_t)blockIdx.x * TILE, tv, TILE);
        __builtin_amdgcn_sched_barrier(0);
    }
    Scratch X = open_call(R);
    if (!server_ends(TILES, MANY, PAIRS)) X.ends = 0;
    const TileRec T = PAIRS ? L.paired_tiles[blockIdx.x] : MIXED ? L.grid_tiles[blockIdx.x] : L.tiles[blockIdx.x];
    if constexpr (PAIRS) {
        if (T.words == TILE_PAIR) {
            __shared__ __align__(16) float more[MANY ? PAIR_EXCHANGE + PAIR_VALUES : SUM_TABLE];
            const unsigned left = server_pair<MANY>(L, A, T, X, set, S, lds, more);
            end_call(left, R, X, S);
            return;
        }
    }
    const int32_t tile = MIXED || PAIRS ? T.tile : (int32_t)blockIdx.x;
    const int64_t tile_start = (int64_t)tile * TILE;
    const int n_valid = MIXED ? tile_valid(L, tile) : TILE;
    float *te = A.err + tile_start;
    unsigned left;
    if (!MIXED || T.words < 0) {
        if (MIXED || PAIRS) {
            load_sign_halves(A, tile_start, 0, h);
            if (MANY) load_sign_halves(A, tile_start, SERVER_CHUNK, h1);
            load_tile(te, tv, TILE);
            __builtin_amdgcn_sched_barrier(0);
        }
        Posted P;
        const BlockSpan sp = span_of(T.bs(), T.be());
        const LoadedCorrection corr = loaded_correction(L, T.fb, X, set);
        correct_loaded_residual(tv, corr);
        server_values_whole<MANY>(A, tile_start, T.fb, h, h1, tv, p, lds);
        const int kind = compress_uniform(p, L, tile, T.fb, sp, TILE, A.signs, A.scales, te, X, set, S, P);
        left = settle_uniform(p, kind, P, tile, T.fb, sp, A.scales, te, L, X, set, S);
    } else if constexpr (MIXED) {
        if (TILES == DENSE_TILES && T.nseg < 0) {
            server_values_mixed(L, A, tile, T, n_valid, te, p, S);
            left = compress_mixed(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S);
            end_call(left, R, X, S);
            return;
        }
        __shared__ FewShared F;
        few_bounds(L, T, tile_start, n_valid, F.bound);
        server_values_few<MANY>(L, A, T, tile_start, te, n_valid, p, lds, F.bound);
        left = compress_few(p, L, T, tile, n_valid, A.signs, A.scales, te, X, set, S, F, lds);
    }
    end_call(left, R, X, S);
}

}  // namespace ef
