// Kernels for launches that (nearly) fit on the GPU all at once: see ef_tile.h for the tile scheme.
//
// A launch of a few hundred tiles is over before HBM or the vector units matter: its time is one
// workgroup's chain of dependent memory round trips (about 0.5 to 1 us each), plus that of every kernel that
// has to follow.  These kernels do the same work as k_worker_tiles / k_server_tiles / k_apply with a shorter
// chain:
//   * what a tile needs to know about both its open blocks comes in one record (SmallTile);
//   * 1024 threads to a tile, four elements each;
//   * all workgroups, or half of them, are resident at once, so all tiles of a block, mixed ones
//     included, can wait for it in place; and they do not wait for a gatherer's answer, each adds up the block's partial
//     sums itself (at most SMALL_SPAN of them: one wavefront, four words a lane);
//   * no kernel follows: the last workgroup to begin steps the call state (see arrive), in a wavefront that has nothing else
//     to do while the others form the block's sum.
#pragma once
#include "ef_layout.h"
#include "ef_tile.h"
#include "ef_worker.h"
#include "ef_server.h"
#include "ef_finish.h"

namespace ef {

constexpr int SMALL_THREADS = 1024;
constexpr int SMALL_WAVES = SMALL_THREADS / 64;
constexpr int COUNT_WAVE = SMALL_WAVES - 1;     // the wavefront that counts the workgroup in

// Up to this many segments of a tile get a wavefront each, of more the short ones get a thread each (server, 4 workers,
// 49 tiles of 64 blocks of 64: 11.4 us a wavefront each, 7.5 a thread each).
constexpr int SMALL_BY_WAVE = 16;

struct SmallTile {
    int32_t fb, nseg;           // first block and number of segments
    int32_t whole;              // inside one block, and not the ragged end of the vector
    int32_t flags;
    int32_t head_t0, head_n;    // tiles of the first segment's block, if it is open (SMALL_HEAD)
    int32_t tail_n;             // tiles of the last segment's block, if that one is (SMALL_TAIL): it starts in this tile
    int32_t unused;
    int64_t head_db, tail_db;   // elements of those blocks
    int16_t bound[SMALL_BY_WAVE + 2];   // of up to SMALL_BY_WAVE segments: where they start, and the last one ends
};
enum {
    SMALL_HEAD = 1,         // the first segment is open (a whole tile has no other)
    SMALL_TAIL = 2,         // the last segment is open, and is not the first
    SMALL_HEAD_SLOT = 4,    // the head block's partial in its first tile is in slot 1 (it starts inside that tile)
    SMALL_WRITES_HEAD = 8,  // this tile is the head block's last: it writes the block's scale
};

struct SmallShared {
    double sum[TILE];           // segment sums; a whole tile: one row sum per thread
    alignas(16) float val[TILE];        // |p| per element
    float scale[TILE];          // segment scales
    int bound[SMALL_BY_WAVE + 1];       // where the segments start, and the last one ends
    int long_list[MAX_LONG];    // of more segments: the ones too long for one thread
    int n_long;
    int parked[2];              // head, tail: the wait ran out
    unsigned park[2];           // as in SyncShared
    unsigned long long own[2];
    unsigned left;              // what arrived() answers
    double total;
};

// What a call reads of the plan.  Everything in it is found by the tile's number, so that nothing but the data waits for the
// record: a scale is two trips to memory away from the kernel's start, not four.
struct SmallTables {
    const SmallTile *tiles;     // [ntiles]
    const StartWord *words;     // [ntiles][TILE_WORDS], whole tiles too; rank: the number of the block in progress before the word, plus 1
    int words_of_tile;          // TILE_WORDS; 0: no tile has two segments, and there is one row of words that nobody looks at
};

// This thread's start word, as it is loaded: looked at only where the segments are wanted, so that nothing else waits for it (its wait
// is one for all that was asked for before it).  No branch: it would end with that wait.
__device__ __forceinline__ StartWord small_word(const SmallTables &Z, int32_t tile)
{
    return Z.words[tile * Z.words_of_tile + (int)(threadIdx.x >> 3)];
}

// This thread's four elements among the blocks.
struct SmallPlace {
    unsigned starts;            // bit c: a segment starts at element c
    int block;                  // the block in progress before element 0 (one before the tile's first: none)
};
__device__ __forceinline__ SmallPlace small_place(const StartWord &w)
{
    SmallPlace q;
    const unsigned sh = (threadIdx.x & 7u) * 4u;
    q.starts = (w.starts >> sh) & 15u;
    q.block = (int)w.rank + __popc(w.starts & ((1u << sh) - 1u)) - 1;
    return q;
}

// Start words by tile, and those of the mixed tiles (k_start_words) on the way (plan creation).  One workgroup of TILE_WORDS
// threads per tile.
__global__ __launch_bounds__(TILE_WORDS) void k_small_words(Layout L, StartWord *words, StartWord *mixed_words)
{
    __shared__ unsigned bits[TILE_WORDS];
    const int32_t tile = blockIdx.x;
    const int64_t tile_start = (int64_t)tile * TILE;
    const int32_t fb = L.tile_fb[tile], lb = L.tile_lb[tile], mixed = L.tiles[tile].words;
    bits[threadIdx.x] = threadIdx.x == 0 ? 1u : 0u;
    __syncthreads();
    for (int32_t b = fb + 1 + (int32_t)threadIdx.x; b <= lb; b += TILE_WORDS) {
        const int j = (int)(L.offs[b] - tile_start);
        atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    unsigned before = 0;
    for (unsigned i = 0; i < threadIdx.x; ++i) before += (unsigned)__popc(bits[i]);
    StartWord w;
    w.starts = bits[threadIdx.x];
    w.rank = before;
    if (mixed >= 0) mixed_words[(int64_t)mixed * TILE_WORDS + threadIdx.x] = w;
    w.rank += (unsigned)fb;
    words[(int64_t)tile * TILE_WORDS + threadIdx.x] = w;
}

__device__ __forceinline__ float4 small_load4(const float *base, int n_valid)
{
    const int j = 4 * (int)threadIdx.x;
    return n_valid == TILE ? stream_load4(base + j) : guarded_load4(base, j, n_valid);
}
__device__ __forceinline__ void small_store4(float *base, int n_valid, float4 v)
{
    const int j = 4 * (int)threadIdx.x;
    if (n_valid == TILE)
        stream_store4(base + j, v);
    else
        guarded_store4(base, j, n_valid, v);
}

// Sign words (as store_signs): 16 lanes make one.
__device__ __forceinline__ void small_signs(float4 p, int n_valid, uint64_t *signs, int64_t tile_start, int64_t W)
{
    const int l16 = lane_id() & 15, j = 4 * (int)threadIdx.x;
    unsigned nib = (p.x >= 0.f ? 1u : 0u) | (p.y >= 0.f ? 2u : 0u) | (p.z >= 0.f ? 4u : 0u) | (p.w >= 0.f ? 8u : 0u);
    if (j + 4 > n_valid) nib &= j < n_valid ? (1u << (n_valid - j)) - 1u : 0u;
    const unsigned sh = (unsigned)(l16 & 7) * 4u;
    unsigned lo = (l16 < 8) ? (nib << sh) : 0u, hi = (l16 >= 8) ? (nib << sh) : 0u;
    lo |= row_move<EF_DPP_XOR1>(lo);
    hi |= row_move<EF_DPP_XOR1>(hi);
    lo |= row_move<EF_DPP_XOR2>(lo);
    hi |= row_move<EF_DPP_XOR2>(hi);
    lo |= row_move<EF_DPP_HALF_MIRROR>(lo);
    hi |= row_move<EF_DPP_HALF_MIRROR>(hi);
    lo |= row_move<EF_DPP_MIRROR>(lo);
    hi |= row_move<EF_DPP_MIRROR>(hi);
    const int64_t w = tile_start / 64 + (threadIdx.x >> 4);
    if (l16 == 0 && w < W) signs[w] = ((uint64_t)hi << 32) | (uint64_t)lo;
}

// The block's partial sums as one wavefront sees them: lane i is in charge of tiles i, i + 64, ...
struct SmallSpan {
    int64_t t0;
    int n, slot;                // slot of the first tile's word
};
__device__ __forceinline__ const unsigned long long *small_part(const unsigned long long *part, const SmallSpan &s, int i)
{
    return part + 2 * (s.t0 + i) + (i == 0 ? s.slot : 0);
}
// The order of sum_block_partials, which has 256 threads.
__device__ __forceinline__ double small_total(const double (&v)[4])
{
    const double a = wave_sum(v[0]), b = wave_sum(v[1]), c = wave_sum(v[2]), d = wave_sum(v[3]);
    return ((a + b) + c) + d;
}
// Waits (bounded) for the partials of all the block's tiles and adds them up.  One wavefront; own: the
// word this workgroup has posted, whose value need not be fetched.
__device__ __forceinline__ bool small_gather(const SmallSpan &s, int own, double own_value, const unsigned long long *part,
                                             unsigned long long tag, int spin_limit, double *total)
{
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    unsigned have = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = lane_id() + 64 * q;
        if (i >= s.n) have |= 1u << q;
        if (i == own) {
            have |= 1u << q;
            v[q] = own_value;
        }
    }
    bool ok = false;
    for (int it = 0; it < spin_limit; ++it) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!((have >> q) & 1u)) {
                const unsigned long long w = __hip_atomic_load(small_part(part, s, lane_id() + 64 * q), __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                if ((w >> 63) == tag) {
                    v[q] = __longlong_as_double((long long)(w & ~TAG_BIT));
                    have |= 1u << q;
                }
            }
        }
        if (__all(have == 15u)) {
            ok = true;
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    if (ok) *total = small_total(v);
    return ok;
}

// Compression of the tile whose values are in p (four consecutive elements a thread): sign words, scales
// of the blocks that end here, e' = p - Delta.  [bs, be): the block of segment threadIdx.x, in a tile of more than SMALL_BY_WAVE.
// COUNTED: the workgroup is counted in (small_arrive), and before is the answer.
template <bool COUNTED>
__device__ __forceinline__ void small_compress(float4 p, const Layout &L, const SmallTile &T,
                                               const StartWord &word, int64_t bs, int64_t be, int n_valid, uint64_t *signs, float *scales_out,
                                               float *err_tile, const Scratch &X, unsigned before, int set, SmallShared &S)
{
    const int32_t tile = blockIdx.x;
    const int lane = lane_id(), wave = wave_id();
    small_signs(p, n_valid, signs, (int64_t)tile * TILE, L.W);
    const int j0 = 4 * (int)threadIdx.x;
    const bool whole = T.whole != 0;
    const double a[4] = {j0 + 0 < n_valid ? fabsf(p.x) : 0.f, j0 + 1 < n_valid ? fabsf(p.y) : 0.f,
                         j0 + 2 < n_valid ? fabsf(p.z) : 0.f, j0 + 3 < n_valid ? fabsf(p.w) : 0.f};
    const unsigned long long tag = set_tag(X, set);
    unsigned long long *part = set_part(X, L, set);
    if (threadIdx.x < 2) {
        S.parked[threadIdx.x] = 0;
        S.own[threadIdx.x] = 0ull;
    }
    if (whole) {
        S.sum[threadIdx.x] = ((a[0] + a[1]) + a[2]) + a[3];
        __syncthreads();
        if (!COUNTED) before = arrive<COUNT_WAVE>(X);
        if (wave == 0) {
            // the order of abs_sum and block_sum: a lane's four rows, the 64 lanes, the four quarters
            double q[4];
#pragma unroll
            for (int w = 0; w < 4; ++w)
                q[w] = ((S.sum[256 * w + lane] + S.sum[256 * w + 64 + lane]) + S.sum[256 * w + 128 + lane]) + S.sum[256 * w + 192 + lane];
            S.total = small_total(q);
        }
    } else {
        // the order of segment_sum
        *reinterpret_cast<float4 *>(&S.val[j0]) = make_float4(fabsf(p.x), fabsf(p.y), fabsf(p.z), fabsf(p.w));
        const int64_t start = (int64_t)tile * TILE;
        if (T.nseg <= SMALL_BY_WAVE) {
            __syncthreads();
            if (!COUNTED) before = arrive<COUNT_WAVE>(X);
#pragma unroll 1
            for (int sg = (int)uniform_u32(threadIdx.x >> 6); sg < T.nseg; sg += SMALL_WAVES) {
                const double total = segment_sum(S.val, (int)uniform_u32((unsigned)S.bound[sg]), (int)uniform_u32((unsigned)S.bound[sg + 1]));
                if (lane == 0) S.sum[sg] = total;
            }
        } else {
            if (threadIdx.x == 0) S.n_long = 0;
            __syncthreads();
            if (!COUNTED) before = arrive<COUNT_WAVE>(X);
            for (int sg = threadIdx.x; sg < T.nseg; sg += SMALL_THREADS) {
                const int64_t b = T.fb + sg;
                const int lo = (int)max((sg < SMALL_THREADS ? bs : L.offs[b]) - start, (int64_t)0);
                const int hi = (int)min((sg < SMALL_THREADS ? be : L.offs[b + 1]) - start, (int64_t)n_valid);
                if (hi - lo > SMALL_SEG) {
                    S.long_list[atomicAdd(&S.n_long, 1)] = sg;
                    continue;
                }
                S.sum[sg] = short_segment_sum(S.val, lo, hi);
            }
            __syncthreads();
            const int n_long = S.n_long;
#pragma unroll 1
            for (int q = (int)uniform_u32(threadIdx.x >> 6); q < n_long; q += SMALL_WAVES) {
                const int sg = S.long_list[q];
                const int64_t b = T.fb + sg;
                const double total = segment_sum(S.val, (int)max(L.offs[b] - start, (int64_t)0), (int)min(L.offs[b + 1] - start, (int64_t)n_valid));
                if (lane == 0) S.sum[sg] = total;
            }
        }
    }
    __syncthreads();
    // the open segments' sums go out first, then the closed segments' scales are formed while others post
    const bool head = T.flags & SMALL_HEAD, tail = T.flags & SMALL_TAIL;
    const double head_sum = whole ? S.total : S.sum[0], tail_sum = whole ? 0.0 : S.sum[T.nseg - 1];
    const SmallSpan hs = {T.head_t0, T.head_n, (T.flags & SMALL_HEAD_SLOT) ? 1 : 0};
    const SmallSpan ts = {tile, T.tail_n, 1};
    if (head) store_partial(head_sum, 0, tile, L, X, set);
    if (tail) store_partial(tail_sum, 1, tile, L, X, set);
    for (int sg = threadIdx.x; sg < T.nseg; sg += SMALL_THREADS) {
        if ((sg == 0 && head) || (sg == T.nseg - 1 && tail)) continue;
        // a closed segment is all of its block
        const int64_t db = whole ? (int64_t)TILE : T.nseg <= SMALL_BY_WAVE ? (int64_t)(S.bound[sg + 1] - S.bound[sg])
                                  : sg < SMALL_THREADS ? be - bs : L.offs[T.fb + sg + 1] - L.offs[T.fb + sg];
        const float sc = (float)((whole ? S.total : S.sum[sg]) / (double)db);
        S.scale[sg] = sc;
        scales_out[T.fb + sg] = sc;
    }
    if ((wave == 0 && head) || (wave == 1 && tail)) {
        const SmallSpan &sp = wave ? ts : hs;
        double total = 0.0;
        const bool ok = small_gather(sp, tile - (int)sp.t0, wave ? tail_sum : head_sum, part, tag, X.spin_limit, &total);
        const int sg = wave ? T.nseg - 1 : 0;
        if (lane == 0) {
            const float sc = (float)(total / (double)(wave ? T.tail_db : T.head_db));
            S.scale[sg] = sc;
            S.parked[wave] = !ok;
            const bool writes = wave == 0 && (T.flags & SMALL_WRITES_HEAD);
            if (ok) {
                if (writes) scales_out[T.fb] = sc;
            } else {
                atomicAdd(X.defer_cnt, 1u);
                if (writes) atomicAdd(X.fin_cnt, 1u);
                give_up(X, &S.park[wave], writes ? PARK_FORMS : 0u);
            }
        }
    }
    // while the others gather; where nothing is gathered, at the end
    if ((head || tail) && wave == COUNT_WAVE) {
        const unsigned left = arrived<COUNT_WAVE>(before, X);
        if (lane == 0) S.left = left;
    }
    __syncthreads();
    const int park_head = S.parked[0], park_tail = S.parked[1];
    const SmallPlace at = small_place(word);
    int seg = T.nseg == 1 ? 0 : at.block - T.fb;
    float v[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        seg += T.nseg == 1 ? 0 : (int)((at.starts >> c) & 1u);
        const float e = residual(v[c], S.scale[seg]);
        const bool keep = (park_head && seg == 0) || (park_tail && seg == T.nseg - 1);
        v[c] = keep ? v[c] : e;
    }
    small_store4(err_tile, n_valid, make_float4(v[0], v[1], v[2], v[3]));
    if (park_head | park_tail) {
        // One wavefront releases for all, whose stores have reached the L2 by then: with a write-back for
        // each, a call whose every wait gives up took 1170 us.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) {
            release_stores();
            if (park_head) leave_entry(S.park[0], 0ull, X, set, tile, 0, &S.own[0]);
            if (park_tail) leave_entry(S.park[1], 0ull, X, set, tile, T.nseg > 1 ? 1 : 0, &S.own[1]);
        }
        __syncthreads();
    }
    if (!(head || tail)) {
        // nothing of its own is left
        if (wave == COUNT_WAVE && arrived<COUNT_WAVE>(before, X)) finish_entries(S.own, false, X);
        return;
    }
    const unsigned left = uniform_u32(S.left);
    // see end_call; all wavefronts are at hand here
    if (left | (unsigned)(park_head | park_tail)) finish_entries(S.own, wave == 0, X);
}

// The bound that this thread puts into SmallShared::bound ahead of small_compress: storing it where it is asked for would wait for all
// that was asked for before it.
__device__ __forceinline__ int small_bound(const SmallTables &Z, int32_t tile)
{
    return Z.tiles[tile].bound[min((int)threadIdx.x, SMALL_BY_WAVE)];
}

__device__ __forceinline__ void put_bound(int bound, SmallShared &S)
{
    if (threadIdx.x <= SMALL_BY_WAVE) S.bound[threadIdx.x] = bound;
}

// Counts the workgroup in as soon as all its wavefronts have the call state in registers: one more barrier, while the tile's
// data are on their way.  Not the server, whose scales wait for the record behind it: it counts behind the first barrier that the sums need
// anyway.  us, here / there: worker of 65 tiles, 4 workers, 7.2 / 7.5, of ResNet-20 7.5 / 7.6; server of ResNet-20 7.5 / 7.2.
__device__ __forceinline__ unsigned small_arrive(const Scratch &X)
{
    asm volatile("" ::"s"(X.tags), "s"(X.epoch), "s"(X.defer_cnt));
    __syncthreads();
    return arrive<COUNT_WAVE>(X);
}

template <bool MOM>
__global__ __launch_bounds__(SMALL_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_worker_small(Layout L, ScratchRef R, WorkerArgs A, SmallTables Z)
{
    __shared__ SmallShared S;
    const int32_t tile = blockIdx.x;
    const int worker = blockIdx.y;
    const int n_valid = tile_valid(L, tile);
    const int64_t start = (int64_t)tile * TILE;
    float *mt = MOM ? A.mom + (int64_t)worker * A.state_stride + start : nullptr;
    float *et = A.err + (int64_t)worker * A.state_stride + start;
    const float4 g = small_load4(A.grad + (int64_t)worker * A.grad_stride + start, n_valid);
    float4 m = g, e = small_load4(et, n_valid);
    if (MOM) m = small_load4(mt, n_valid);
    const StartWord place = small_word(Z, tile);
    const int bound = small_bound(Z, tile);
    const SmallTile T = Z.tiles[tile];
    const Scratch X = open_call(R);
    const unsigned before = small_arrive(X);
    int64_t bs = 0, be = 1;
    if (T.nseg > SMALL_BY_WAVE && (int)threadIdx.x < T.nseg) {
        bs = L.offs[T.fb + threadIdx.x];
        be = L.offs[T.fb + threadIdx.x + 1];
    }
    worker_values4<MOM>(g, m, e, A.mu, A.r);
    if (MOM) small_store4(mt, n_valid, m);
    put_bound(bound, S);
    small_compress<true>(e, L, T, place, bs, be, n_valid, A.signs + (int64_t)worker * A.signs_stride,
                   A.scales + (int64_t)worker * A.scales_stride, et, X, before, worker, S);
}

constexpr int SMALL_CHUNK = 8, SMALL_GROUP = 4;     // workers whose sign words are in flight together, and are added up together
constexpr int SMALL_STAGE = 2 * TILE;       // scales that fit where the sums will be

// Half-word hw of workers i0 .. i0 + 7 (past M: the last worker's again; of a group without any none).
__device__ __forceinline__ void small_words(const ServerArgs &A, int i0, unsigned hw, uint32_t (&word)[SMALL_CHUNK])
{
#pragma unroll
    for (int g = 0; g < SMALL_CHUNK; g += SMALL_GROUP)
        if (g == 0 || i0 + g < A.M)
#pragma unroll
            for (int u = g; u < g + SMALL_GROUP; ++u)
                word[u] = reinterpret_cast<const uint32_t *>(A.signs_in + (int64_t)min(i0 + u, A.M - 1) * A.in_signs_stride)[hw];
}

// The scales of the tile's segments from all workers come in one trip to memory, a wavefront to a worker, and are looked up
// in LDS; one segment's are scalars.  (Gathered by element, four workers at a time, each group waited for the one before it, and
// all of them for the start words, these for the record.  Server call, 16 workers, 322 tiles in blocks of eight
// 14.1 -> 12.6 us; 4 workers, a bottleneck network of 341 tiles 10.2 -> 9.4; 1 worker, 213 tiles 7.4 -> 7.3.)
__global__ __launch_bounds__(SMALL_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_server_small(Layout L, ScratchRef R, ServerArgs A, SmallTables Z, int set)
{
    __shared__ SmallShared S;
    const int32_t tile = blockIdx.x;
    const int n_valid = tile_valid(L, tile);
    const int64_t start = (int64_t)tile * TILE;
    float *et = A.err + start;
    const float4 te = small_load4(et, n_valid);
    const StartWord place = small_word(Z, tile);
    const int bound = small_bound(Z, tile);
    // this thread's four sign bits are in one half-word of every payload (past the end: elements that are not stored)
    const unsigned last = (unsigned)(2 * L.W - 1), hw = min((unsigned)(start >> 5) + (threadIdx.x >> 3), last);
    const unsigned sh = (threadIdx.x & 7u) * 4u;
    uint32_t word[SMALL_CHUNK];
    small_words(A, 0, hw, word);
    const SmallTile T = Z.tiles[tile];
    const Scratch X = open_call(R);
    int64_t bs = 0, be = 1;
    if (T.nseg > SMALL_BY_WAVE && (int)threadIdx.x < T.nseg) {
        bs = L.offs[T.fb + threadIdx.x];
        be = L.offs[T.fb + threadIdx.x + 1];
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (T.nseg == 1) {
#pragma unroll 1
        for (int i0 = 0; i0 < A.M; i0 += SMALL_CHUNK) {
            float sc[SMALL_CHUNK];
            // vector loads: the eight scalar ones of load_scales took 0.5 us more (server call, 1 worker, 392 tiles 8.6 -> 8.0)
            unsigned zero = 0u;
            asm("" : "+v"(zero));
#pragma unroll
            for (int g = 0; g < SMALL_CHUNK; g += SMALL_GROUP)
                if (g == 0 || i0 + g < A.M)
#pragma unroll
                    for (int u = g; u < g + SMALL_GROUP; ++u)
                        sc[u] = A.scales_in[(int64_t)min(i0 + u, A.M - 1) * A.in_scales_stride + T.fb + zero];
            if (i0 > 0) small_words(A, i0, hw, word);
#pragma unroll
            for (int g = 0; g < SMALL_CHUNK; g += SMALL_GROUP)
                if (g == 0 || i0 + g < A.M)
#pragma unroll
                    for (int u = g; u < g + SMALL_GROUP; ++u)
                        if (i0 + u < A.M)
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[c] = acc[c] + signed_scale(sc[u], (word[u] >> (sh + c)) & 1u);
        }
        put_bound(bound, S);
    } else {
        int seg[4];
        const auto segments = [&] {
            const SmallPlace at = small_place(place);
            int sg = at.block - T.fb;
#pragma unroll
            for (int c = 0; c < 4; ++c) seg[c] = sg += (int)((at.starts >> c) & 1u);
        };
        float *stage = reinterpret_cast<float *>(S.sum);
        const int rows = (A.M + SMALL_GROUP - 1) / SMALL_GROUP * SMALL_GROUP;
        if (T.nseg * rows <= SMALL_STAGE) {
#pragma unroll 1
            for (int u = wave_id(); u < rows; u += SMALL_WAVES) {
                const float *sc = A.scales_in + (int64_t)min(u, A.M - 1) * A.in_scales_stride + T.fb;
#pragma unroll 1
                for (int j = lane_id(); j < T.nseg; j += 64) stage[u * T.nseg + j] = u < A.M ? sc[j] : 0.0f;
            }
            put_bound(bound, S);
            __syncthreads();
            segments();
#pragma unroll 1
            for (int i0 = 0; i0 < A.M; i0 += SMALL_CHUNK) {
                if (i0 > 0) small_words(A, i0, hw, word);
#pragma unroll
                for (int g = 0; g < SMALL_CHUNK; g += SMALL_GROUP)
                    if (g == 0 || i0 + g < A.M)
#pragma unroll
                        for (int u = g; u < g + SMALL_GROUP; ++u)
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                acc[c] = acc[c] + signed_scale(stage[seg[c]], (word[u] >> (sh + c)) & 1u);
                                seg[c] += T.nseg;
                            }
            }
        } else {
            // more segments than the stage holds: a gather for each element
            segments();
#pragma unroll 1
            for (int i = 0; i < A.M; ++i) {
                const float *sc = A.scales_in + (int64_t)i * A.in_scales_stride + T.fb;
                const uint32_t w = reinterpret_cast<const uint32_t *>(A.signs_in + (int64_t)i * A.in_signs_stride)[hw];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] = acc[c] + signed_scale(sc[seg[c]], (w >> (sh + c)) & 1u);
            }
        }
        __syncthreads();            // the stage is read no more
    }
    float4 p;
    p.x = mean_of(acc[0], A.Mf, A.Minv) + A.r * te.x;
    p.y = mean_of(acc[1], A.Mf, A.Minv) + A.r * te.y;
    p.z = mean_of(acc[2], A.Mf, A.Minv) + A.r * te.z;
    p.w = mean_of(acc[3], A.Mf, A.Minv) + A.r * te.w;
    small_compress<false>(p, L, T, place, bs, be, n_valid, A.signs, A.scales, et, X, 0u, set, S);
}

// Parameter update (see apply_tile), one workgroup of 1024 threads per tile.
template <bool WD>
__global__ __launch_bounds__(SMALL_THREADS) void k_apply_small(ApplyTables Z, float *x, float *mt, const uint64_t *signs,
                                                               const float *scales, float eta, float mu, float lambda)
{
    const int32_t tile = blockIdx.x;
    const int n_valid = tile_valid(Z.d, tile);
    const int64_t start = (int64_t)tile * TILE;
    const int64_t last = 2 * Z.W - 1, hw = (start >> 5) + (threadIdx.x >> 3);
    StartWord place = {0u, 0u};
    if (Z.words) place = Z.words[tile * TILE_WORDS + (int)(threadIdx.x >> 3)];
    const uint32_t word = reinterpret_cast<const uint32_t *>(signs)[hw < last ? hw : last];
    const float4 x4 = small_load4(x + start, n_valid);
    float4 m4 = x4;
    if (WD) m4 = small_load4(mt + start, n_valid);
    float xv[4] = {x4.x, x4.y, x4.z, x4.w}, mv[4] = {m4.x, m4.y, m4.z, m4.w};
    const SmallPlace at = small_place(place);
    int block = Z.words ? at.block : Z.tiles[tile].fb;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        block += (int)((at.starts >> c) & 1u);
        const float delta = signed_scale(scales[block], (word >> ((threadIdx.x & 7u) * 4u + c)) & 1u);
        update_element<WD>(xv[c], mv[c], delta, eta, mu, lambda);
    }
    small_store4(x + start, n_valid, make_float4(xv[0], xv[1], xv[2], xv[3]));
    if (WD) small_store4(mt + start, n_valid, make_float4(mv[0], mv[1], mv[2], mv[3]));
}

}  // namespace ef
