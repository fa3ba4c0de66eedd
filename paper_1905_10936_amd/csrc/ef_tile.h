// Device side of libef: tile-based kernels for the worker, server and apply
// steps of Algorithm 4 (dist-EF-blockSGDM, arxiv 1905.10936), written for
// gfx950 (64-lane wavefronts, 256 CUs in 8 XCDs, HBM-bound streaming passes).
//
// Work decomposition
// ------------------
// The flat d-vector is cut into tiles of TILE = 4096 consecutive elements, the
// unit of work of a 256-thread workgroup.  Tiles, not blocks, are the unit, so
// a block of 8M elements and a block of 1 element cost the same per element.
// A tile is a whole number of 64-element sign words and starts on a 16 KiB
// boundary, so every fp32 access is a coalesced 128-bit access whatever the
// block boundaries are.  Inside a tile, wavefront w owns the 1024 consecutive
// elements [1024w, 1024w+1024) as 4 sub-rows of 256; lane l of sub-row k holds
// the 4 consecutive elements 1024w + 256k + 4l .. +3.
//
// The blocks of the partition (Section 3.2) cut a tile into segments.  A full
// tile that lies inside one block is "uniform"; a tile where several blocks
// meet, and the ragged last tile of the vector, is "mixed".  A segment whose block lies entirely inside the tile is "closed":
// its L1 norm, scale and residual are finished by the tile alone (in fp64, in
// the one order of segment_sum).  The other segments are "open": their
// fp64 partial sums go to a per-(tile, slot) scratch word, and whoever needs
// the block's scale adds the block's partials in one fixed order (thread t
// takes tiles t, t+256, ... ascending, then a fixed tree), so the scale has the
// same bits wherever and whenever it is computed.
//
// One pass over the state
// -----------------------
// e <- p - Delta needs the block's scale, i.e. every tile of the block.  For a
// block of at most `fuse_limit` tiles the workgroups of its uniform tiles keep
// p in registers until the scale exists and then write the finished residual,
// so every fp32 tensor is read once and written once.  The hand-off between
// workgroups uses relaxed agent-scope atomics only (an agent-scope release
// fence would write back the whole L2 of streaming stores on every tile):
//   * a partial is never negative, so its sign bit carries a tag that flips on
//     every call that uses the scratch set; one 64-bit store publishes value
//     and tag together;
//   * the workgroup that takes the block's last whole tile gathers the
//     partials (re-reading those whose tag is still old: tiles are handed out
//     in ascending order, so the others are at most a tile-time behind),
//     writes the scale and posts (call number, scale) in the block's "ready"
//     word -- no counter, hence no read-modify-write on a shared address;
//   * the others look at the ready word when they come to write the tile.
// The kernels that run one workgroup per tile take the mixed tiles of a few
// segments in their place among the whole ones, and their open segments wait like
// whole tiles do.  The "dense" ones, of many segments, come first in their grid, and before the
// persistent worker kernel all mixed tiles run in a kernel of their own,
// so their partial sums are there when a block's last whole tile comes to form the
// scale; they never wait for a whole tile: a block without whole tiles is
// finished among them (its last tile forms its scale, the
// others wait for it), while the segments that a block with whole tiles has in
// them get p parked in the residual buffer.  Parked p (those segments, the
// tiles of blocks larger than fuse_limit but for the last ones (first_kept), any tile whose bounded wait ran out) is finished by one kernel
// after the main one, which also computes the scales still missing and steps
// the plan to its next call.  Where a layout leaves nothing to that kernel but the last two, the main one sees to them (see
// ARRIVE_GROUPS).
//
// Deferred correction (optional)
// ------------------------------
// With Layout::lazy set, the whole tiles of blocks larger than fuse_limit are
// left out of that last kernel: the buffer keeps p, the block's scale is kept
// in Scratch::lazy_scales, a bit per set in CallState says so, and the next
// call subtracts the decoded value as it loads the tile (loaded_correction).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "ef_layout.h"

namespace ef {

constexpr int TILE = 4096;      // elements per workgroup and step
constexpr int THREADS = 256;    // 4 wavefronts
constexpr int NWAVES = THREADS / 64;
constexpr int SUBROWS = 4;      // float4 per thread
constexpr int SMALL_SEG = 64;   // segments up to this length are summed by one thread
constexpr int MAX_LONG = TILE / SMALL_SEG;
constexpr int TILE_WORDS = TILE / 32;
constexpr int DEFER_WGS = 16;   // workgroups that serve the run-time lists in the kernel that ends a call
constexpr int FIN_WGS_MAX = 512;    // most workgroups that kernel gives to the scales of blocks larger than fuse_limit ...
constexpr int RES_WGS_MAX = 2048;   // ... and to the segments whose p was parked
constexpr int RES_IN_TAIL_MAX = 4 * RES_WGS_MAX;    // longer lists of parked segments get a kernel of their own
#ifndef EF_PIPE_DEPTH
#define EF_PIPE_DEPTH 3
#endif
constexpr int PIPE_DEPTH = EF_PIPE_DEPTH;     // tiles a persistent workgroup keeps in registers while their scales form
constexpr unsigned long long TAG_BIT = 1ull << 63;
constexpr int FUSE_LIMIT_MAX = 4096;                     // most tiles a one-pass block may be given through ef_plan_tune

// What the kernels need to know about a tile, in one record: looked up piece by piece (tile, its block, the
// block's ends) it is three dependent loads before the first scale can be asked for, and two more between
// a tile's sum and its posting.
constexpr int32_t TILE_ALONE = -1, TILE_PAIR = -2;
struct alignas(32) TileRec {
    int32_t tile;
    int32_t fb;                 // first block
    int32_t nseg;               // segments; < 0: that many, and the tile is a dense one
    int32_t words;              // < 0: a whole tile (TILE_PAIR: it and the next one); else which set of start words (its place among the mixed tiles)
    int32_t tail;               // 0, or, if the last of several segments goes on past the tile: its block's tiles * 2,
                                // + 1 if the block ends inside its last tile
    int32_t t0, n;              // tiles of the first block
    int16_t from, to;           // where it starts in its first tile, and ends in its last (0: at the tile's end)
    __host__ __device__ int64_t bs() const { return (int64_t)t0 * TILE + from; }
    __host__ __device__ int64_t be() const { return (int64_t)(t0 + n - 1) * TILE + (to ? to : TILE); }
};
// Where the segments of a mixed tile start, 32 elements to a word; written at plan creation.
struct StartWord {
    uint32_t starts;            // bit j: a segment starts at element j of the 32 (the tile's first always does)
    uint32_t rank;              // starts before the word
};

struct Layout {
    int64_t d;                  // elements
    int64_t B;                  // blocks
    int64_t W;                  // sign words
    int32_t ntiles;
    int32_t fuse_limit;         // blocks of up to this many tiles finish in one pass
    int32_t keep;               // of larger ones about this many of the last whole tiles do too (see first_kept); 0: none
    int32_t n_mixed, n_uniform;
    const int64_t *offs;        // [B+1] device copy of block_offsets
    const int32_t *tile_fb;     // [ntiles] block holding the tile's first element
    const int32_t *tile_lb;     // [ntiles] block holding the tile's last valid element
    const int32_t *mixed_tiles;   // [n_mixed] ascending
    const TileRec *mixed_recs;    // [n_mixed] the same
    const int32_t *whole_tiles;   // [n_uniform] ascending
    const TileRec *tiles;         // [ntiles]
    int32_t n_grid;
    const TileRec *grid_tiles;    // [n_grid] as the kernels with one workgroup per tile take them: the dense ones first
    int32_t n_paired;
    const TileRec *paired_tiles;  // [n_paired] the same for k_server_tiles with two whole tiles to a workgroup
    const StartWord *words;       // [n_mixed][TILE_WORDS]
    int32_t n_dense;              // mixed tiles of many segments
    // Deferred correction (see Scratch::lazy_scales): on or off, and for every block its position
    // among the blocks larger than fuse_limit (-1 for the others).
    int32_t lazy;
    const int32_t *late_index;    // [B]
    // Whole tiles of blocks larger than fuse_limit are written out in groups of this many
    // consecutive tiles (see sync_group_wait); 0 or 1: every tile on its own.
    int32_t sync_group;
};

// What changes from call to call lives in device memory, so that the kernel
// arguments of a call are the same every time (a captured HIP graph of the
// calls can be replayed): the number of calls made on the plan and the tag each
// scratch set's partial words carry since the last call that used the set.
// Whoever ends a call moves it on: the last workgroup of the main kernel to begin (arrived), or k_tail, whose own
// workgroups go by the copy that the call's main kernel leaves in ScratchRef::snapshot, so nothing has to wait for them.
struct alignas(32) CallState {
    unsigned int calls;
    unsigned int server_tag;            // bit 0
    unsigned long long worker_tags;     // bit i: worker i
    unsigned long long worker_pending;  // bit i: worker i's residual buffer holds uncorrected p in its large blocks
    unsigned int server_pending;        // bit 0: the same for the server residual
};

// A call whose main kernel leaves nothing for certain to another one ends without k_tail (ScratchRef::ends).  Every workgroup
// counts itself in once it has read the call state, on one of ARRIVE_GROUPS words a cache line apart; the last of a group
// counts the group on one word more, and the last of all steps the call state: nobody reads it any more.  The count's answer
// comes back while the workgroup waits for its block's scale, so that it costs no time.  (Counting out at the end does: an atomic's answer takes several us while HBM is saturated.)
// A wait that runs out goes by the same word.  The workgroup leaves p in the residual buffer.  If all workgroups have begun, all
// partial sums are sure to come (each posts its own ahead of its waits), and it waits for them at its end and finishes the
// segment.  Else it is counted there as parked and leaves an entry in ScratchRef::parked.  The last workgroup to begin finds the
// number of entries in its own count's answer and sees to them, and others that are at hand with it (finish_entries).
constexpr int ARRIVE_GROUPS = 32, ARRIVE_STRIDE = 32;       // words
constexpr int ARRIVE_AT = 32;                               // the first of them, after a parity's counters (ScratchRef::list_cnt)
constexpr int LEFT = ARRIVE_GROUPS + 1;                     // after the count's words: number of entries and 1, when all have begun
constexpr int TAKEN = LEFT + 1;                             // and of those that somebody sees to
constexpr int CALL_WORDS = ARRIVE_AT + (TAKEN + 1) * ARRIVE_STRIDE;
constexpr unsigned ARRIVED_MASK = 255u, PARKED_ONE = 256u;  // on the last word: groups that are complete; parked entries
constexpr int64_t ENDS_WGS_MAX = 1 << 16;                   // workgroups of such a call: of more, k_tail's 5 us are nothing
constexpr unsigned PARK_FORMS = 1u << 31;                   // the same beside an entry's number (SyncShared::park)
constexpr unsigned PARK_OWN = PARK_FORMS - 1u;              // in place of the number: the workgroup's own to see to

// Kernel argument: the plan's scratch.  A "set" is one worker, or the server.
struct ScratchRef {
    unsigned long long *part;
    unsigned long long *ready;
    unsigned long long *defer_list;
    unsigned long long *fin_list;
    unsigned int *list_cnt;             // [CALL_WORDS]: defer_cnt[2], fin_cnt[2], ticket[2], lost_cnt[2], then the words of the
                                        // count of workgroups, two each (a call uses those of its parity)
    float *lazy_scales;                 // [nsets][lazy_stride] last scale of every block larger than fuse_limit
    int lazy_stride;
    const CallState *state;
    CallState *snapshot;                // what the call's main kernel found in *state, for the kernel that ends the call
    int set_base;                       // first set this call uses (0 for workers, max_workers for the server)
    int spin_limit;
    // of a call that ends without k_tail
    int ends;
    int columns, nsets;                 // workgroups: of a set, and sets
    int lazy;
    CallState *step;
    unsigned long long *parked;         // entries (parked_entry), all 0 between calls but for what was lost
    float *err;                         // residual buffers of the call's sets, err_stride apart
    int64_t err_stride;
    float *scales;                      // scale arrays of the call's sets, scales_stride apart
    int64_t scales_stride;
};

// The arguments every kernel that may end its call begins with, read again where they are seldom needed: kept from the
// kernel's start they cost it scalar registers throughout.
struct CallArgs {
    Layout L;
    ScratchRef R;
};
__device__ __forceinline__ const CallArgs &call_args()
{
    typedef __attribute__((address_space(4))) const void *Segment;
    Segment at = (Segment)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const CallArgs *)at;
}

// Scratch of one call, formed by every kernel from ScratchRef and CallState (open_call).
struct Scratch {
    unsigned long long *part;   // [nsets][2*ntiles] tagged fp64 partial sums of open segments
    unsigned long long *ready;  // [nsets][ntiles][READY_STRIDE]: (epoch << 32) | scale bits in the line of the block's gatherer tile
    unsigned int *defer_cnt;    // entries in defer_list for this call
    unsigned long long *defer_list;  // parked segments: (set << 33) | (tile << 1) | slot
    unsigned int *fin_cnt;      // entries in fin_list for this call
    unsigned long long *fin_list;    // blocks whose scale is still to be written: (set << 32) | block
    unsigned int *ticket;       // next chunk of tiles to hand out (persistent kernels), 0 at call start
    unsigned long long tags;    // bit i = this call's tag of set (set_base + i), carried by its partial words
    unsigned int epoch;         // this call's number on the plan (never 0), carried by the ready words
    int set_base;               // first set this call uses (0 for workers, max_workers for the server)
    int spin_limit;             // polls before a waiting workgroup gives up and parks p
    unsigned int *lost_cnt;     // waits of a group (sync_group_wait) that ran out in this call: a diagnostic
    unsigned int *next_cnt;     // the counters of the next call (zeroed by whoever ends this one)
    int ends;                   // the call ends without k_tail
    // Deferred correction.  A block larger than fuse_limit cannot have its residual finished in
    // the first kernel; instead of a second pass over it (p written, read back, e written: 8 more
    // bytes per element), the residual buffer keeps p, the block's scale is remembered here, and
    // the next call that loads the buffer subtracts the decoded value on the fly: the same fp32
    // operation on the same operands, one call later.  `pending` says for which sets that is due.
    float *lazy_scales;
    int lazy_stride;
    unsigned long long pending;  // bit i: set (set_base + i)
};

__device__ __forceinline__ unsigned uniform_u32(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v)
{
    return ((unsigned long long)uniform_u32((unsigned)(v >> 32)) << 32) | uniform_u32((unsigned)v);
}

// Every workgroup's first dependent load, ahead of anything it can ask for by tile: the whole record in one scalar
// load and no branch between it and what follows.
__device__ __forceinline__ Scratch open_call(const ScratchRef &R)
{
    Scratch X;
    const CallState now = *R.state;
    const unsigned calls = uniform_u32(now.calls);
    const unsigned long long worker_tags = uniform_u64(now.worker_tags), worker_pending = uniform_u64(now.worker_pending);
    const unsigned server_tag = uniform_u32(now.server_tag), server_pending = uniform_u32(now.server_pending);
    const bool workers = R.set_base == 0;
    const unsigned cur = calls & 1u;
    X.part = R.part;
    X.ready = R.ready;
    X.defer_list = R.defer_list;
    X.fin_list = R.fin_list;
    X.defer_cnt = R.list_cnt + cur;
    X.fin_cnt = R.list_cnt + 2 + cur;
    X.ticket = R.list_cnt + 4 + cur;
    X.lost_cnt = R.list_cnt + 6 + cur;
    X.next_cnt = R.list_cnt + (cur ^ 1u);
    // this call's tags are the stored ones flipped
    X.tags = workers ? ~worker_tags : (unsigned long long)(server_tag ^ 1u);
    X.lazy_scales = R.lazy_scales;
    X.lazy_stride = R.lazy_stride;
    X.pending = workers ? worker_pending : (unsigned long long)(server_pending & 1u);
    X.epoch = calls % 0xffffffffu + 1u;     // never 0: 0 marks "no scale posted"
    X.set_base = R.set_base;
    X.spin_limit = R.spin_limit;
    X.ends = R.ends;
    return X;
}

// The call's main kernel leaves what it goes by for the kernel that ends the call.  Called at the main
// kernel's end: a store ahead of the loads of scales and block offsets keeps the compiler from making
// them scalar loads (measured: server call with 16 workers 1.12 -> 1.26 ms).
__device__ __forceinline__ void snapshot_call(const ScratchRef &R)
{
    if (!R.ends && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *R.snapshot = *R.state;
}

struct WorkerArgs {
    const float *grad; int64_t grad_stride;
    float *mom; float *err; int64_t state_stride;
    float mu, r;
    uint64_t *signs; float *scales;
    int64_t signs_stride;       // 64-bit words between the payloads of two workers
    int64_t scales_stride;      // floats between the scale arrays of two workers
};

struct ServerArgs {
    int M;
    const uint64_t *signs_in;   // worker i at signs_in + i*in_signs_stride (64-bit words)
    const float *scales_in;     // worker i at scales_in + i*in_scales_stride (floats)
    int64_t in_signs_stride, in_scales_stride;
    float *err;                 // server residual
    float r, Mf;
    float Minv;                 // 1/M if M is a power of two (exact), else 0
    uint64_t *signs; float *scales;
};

// ---------------------------------------------------------------- helpers ---

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }
// first local element of this thread's float4 in sub-row k
__device__ __forceinline__ int local_base(int k) { return wave_id() * 1024 + k * 256 + lane_id() * 4; }

// The fp32 state is streamed: each element is read once and written once per
// call, so loads and stores carry the non-temporal hint and do not displace
// the little that is reused (offsets, scales, partial sums) from the caches.
typedef float vf4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 stream_load4(const float *p)
{
    const vf4 v = __builtin_nontemporal_load(reinterpret_cast<const vf4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void stream_store4(float *p, float4 a)
{
    const vf4 v = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(v, reinterpret_cast<vf4 *>(p));
}

// Past the end: the last element again, which whoever uses the values leaves out (sums and sign words go by n_valid,
// stores are guarded).  Putting zeros there here made every group wait for its own loads, one after the other: a
// call's one ragged tile was what a small call waited for (update with weight decay, 16 tiles: 5.2 us, 3.1 without it).
__device__ __forceinline__ float4 guarded_load4(const float *base, int local, int n_valid)
{
    const int last = n_valid - 1;
    return make_float4(base[min(local, last)], base[min(local + 1, last)], base[min(local + 2, last)], base[min(local + 3, last)]);
}

__device__ __forceinline__ void guarded_store4(float *base, int local, int n_valid, float4 v)
{
    if (local + 0 < n_valid) base[local + 0] = v.x;
    if (local + 1 < n_valid) base[local + 1] = v.y;
    if (local + 2 < n_valid) base[local + 2] = v.z;
    if (local + 3 < n_valid) base[local + 3] = v.w;
}

template <class T>
__device__ __forceinline__ T *tile_part(T *base, int k)
{
    unsigned at = (threadIdx.x >> 6) * 4096u + (threadIdx.x & 63u) * 16u;
    asm("" : "+v"(at));
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type C;
    return reinterpret_cast<T *>(reinterpret_cast<C *>(base) + at) + k * 256;
}

// A thread's four float4 of one tile.  Only the last tile of a vector can be
// ragged; the test is uniform over the workgroup, so full tiles run straight
// through 128-bit accesses with no per-access branch.
__device__ __forceinline__ void load_tile(const float *base, float4 (&v)[SUBROWS], int n_valid)
{
    if (n_valid == TILE) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) v[k] = stream_load4(tile_part(base, k));
    } else {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) {
            v[k] = guarded_load4(base, local_base(k), n_valid);
            __builtin_amdgcn_sched_barrier(0);      // addresses one group after the other: few registers
        }
    }
}

__device__ __forceinline__ void clear_past_end(float4 (&v)[SUBROWS], int n_valid)
{
    if (n_valid == TILE) return;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        const int j = local_base(k);
        v[k].x = j + 0 < n_valid ? v[k].x : 0.f;
        v[k].y = j + 1 < n_valid ? v[k].y : 0.f;
        v[k].z = j + 2 < n_valid ? v[k].z : 0.f;
        v[k].w = j + 3 < n_valid ? v[k].w : 0.f;
    }
}

__device__ __forceinline__ void store_tile(float *base, const float4 (&v)[SUBROWS], int n_valid)
{
    if (n_valid == TILE) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) stream_store4(tile_part(base, k), v[k]);
    } else {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) guarded_store4(base, local_base(k), n_valid, v[k]);
    }
}

__device__ __forceinline__ int tile_valid(int64_t d, int32_t tile)
{
    const int64_t left = d - (int64_t)tile * TILE;
    return left >= TILE ? TILE : (int)left;
}
__device__ __forceinline__ int tile_valid(const Layout &L, int32_t tile) { return tile_valid(L.d, tile); }

// Data-parallel-primitive moves inside a row of 16 lanes: the value of the lane
// whose index differs in bit 0 / bit 1, and of the mirror lane within 8 / 16
// lanes.  Applied in this order to an associative, commutative operation they
// leave its result over the whole row in every lane of the row (after the
// first two steps a group of four lanes agrees, and the mirrors pair up whole
// groups), with no LDS traffic.
#define EF_DPP_XOR1 0xB1            // quad_perm [1,0,3,2]
#define EF_DPP_XOR2 0x4E            // quad_perm [2,3,0,1]
#define EF_DPP_HALF_MIRROR 0x141    // lane i <- lane 7-i of its group of 8
#define EF_DPP_MIRROR 0x140         // lane i <- lane 15-i of its row
#define EF_DPP_FROM_4_ON 0x104      // lane i <- lane i+4 of its row (0 past the row)
#define EF_DPP_FROM_8_ON 0x108      // lane i <- lane i+8
template <int CTRL>
__device__ __forceinline__ unsigned row_move(unsigned v)
{
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double row_move(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = row_move<CTRL>((unsigned)b), hi = row_move<CTRL>((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// v of this lane plus v of the lane whose index differs in bit 4 (WIDTH = 16) or bit 5 (32).  The swap leaves both
// rows' values in every lane of the pair of rows, in one instruction per half of the number and without LDS.
template <int WIDTH>
__device__ __forceinline__ double add_other_row(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
    typedef unsigned vu2 __attribute__((ext_vector_type(2)));
    vu2 l, h;
    if constexpr (WIDTH == 16) {
        l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    } else {
        l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    }
    return __longlong_as_double((long long)(((unsigned long long)h.x << 32) | l.x)) +
           __longlong_as_double((long long)(((unsigned long long)h.y << 32) | l.y));
}

// Sum over the 64 lanes in a fixed order: every lane ends with the same bits.
__device__ __forceinline__ double wave_sum(double v)
{
    v += row_move<EF_DPP_XOR1>(v);
    v += row_move<EF_DPP_XOR2>(v);
    v += row_move<EF_DPP_HALF_MIRROR>(v);
    v += row_move<EF_DPP_MIRROR>(v);
    v = add_other_row<16>(v);
    return add_other_row<32>(v);
}

// Sum of val[j], val[j + STEP], ... below hi, one after the other, on top of acc.  The reads go out eight at a time;
// adding the +0 that stands for one past the end changes nothing, since no element is negative.
template <int STEP>
__device__ __forceinline__ double ordered_sum(const float *val, int j, int hi, double acc)
{
#pragma unroll 1
    for (; j + 7 * STEP < hi; j += 8 * STEP) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = val[j + q * STEP];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += (double)v[q];
    }
    if (j + 3 * STEP < hi) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = val[j + q * STEP];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += (double)v[q];
        j += 4 * STEP;
    }
    if (j < hi) {
        float v[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = val[min(j + q * STEP, hi - 1)];
#pragma unroll
        for (int q = 0; q < 3; ++q) acc += (double)(j + q * STEP < hi ? v[q] : 0.f);
    }
    return acc;
}

// Sum of val[lo], ..., val[hi - 1] ascending, by one thread, with 128-bit reads (val is 16-byte aligned): many threads
// read at once, and segments of one length share banks (ef_small.h, server call on
// 49 tiles of blocks of 64: 7.5 us, 8.6 with 32-bit reads).
__device__ __forceinline__ double short_segment_sum(const float *val, int lo, int hi)
{
    int j = lo & ~3;
    double acc;
    {
        const float4 v = *reinterpret_cast<const float4 *>(val + j);
        acc = (double)(j >= lo ? v.x : 0.f);
        acc += (double)(j + 1 >= lo && j + 1 < hi ? v.y : 0.f);
        acc += (double)(j + 2 >= lo && j + 2 < hi ? v.z : 0.f);
        acc += (double)(j + 3 < hi ? v.w : 0.f);
        j += 4;
    }
#pragma unroll 1
    for (; j + 8 <= hi; j += 8) {
        const float4 v = *reinterpret_cast<const float4 *>(val + j), w = *reinterpret_cast<const float4 *>(val + j + 4);
        acc += (double)v.x;
        acc += (double)v.y;
        acc += (double)v.z;
        acc += (double)v.w;
        acc += (double)w.x;
        acc += (double)w.y;
        acc += (double)w.z;
        acc += (double)w.w;
    }
#pragma unroll 1
    for (; j < hi; j += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(val + j);
        acc += (double)v.x;
        acc += (double)(j + 1 < hi ? v.y : 0.f);
        acc += (double)(j + 2 < hi ? v.z : 0.f);
        acc += (double)(j + 3 < hi ? v.w : 0.f);
    }
    return acc;
}

// Sum of |p| over the segment [lo, hi) of a tile, val: |p| of the tile's elements, in LDS.  THE order, whichever kernel
// forms it, so that a block's scale has the same bits on every route: up to SMALL_SEG elements ascending; else lane l
// adds lo + l, lo + l + 64, ... and the lanes are added up by wave_sum.  One wavefront, lo and hi the same in all
// lanes; every lane gets the sum.
__device__ __forceinline__ double segment_sum(const float *val, int lo, int hi)
{
    if (hi - lo > SMALL_SEG) return wave_sum(ordered_sum<64>(val, lo + lane_id(), hi, 0.0));
    return ordered_sum<1>(val, lo, hi, 0.0);        // one address for all lanes: one access
}

// Workgroup sum in a fixed order; every thread gets the same bits.
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    if (lane_id() == 0) red[wave_id()] = v;
    __syncthreads();
    double t = ((red[0] + red[1]) + red[2]) + red[3];
    __syncthreads();
    return t;
}

// value the payload stands for: +s if bit else -s (negation is exact)
__device__ __forceinline__ float signed_scale(float s, bool plus) { return plus ? s : -s; }
// e' = p - Delta for one element whose block has scale s
__device__ __forceinline__ float residual(float p, float s) { return p - signed_scale(s, p >= 0.f); }

__device__ __forceinline__ void residual4(float4 &v, float s)
{
    v.x = residual(v.x, s);
    v.y = residual(v.y, s);
    v.z = residual(v.z, s);
    v.w = residual(v.w, s);
}

// Sign bits (bit = p >= 0, Appendix A with sign(0) read as +1; elements past n_valid give 0 bits) of a quarter of a tile,
// 1024 elements a wavefront: this lane's 16 of them, elements 256 (lane % 4) + 16 (lane / 4) on.  A lane's 16 bits are four from each of its
// sub-rows; four neighbouring lanes transpose their 4 x 4 nibbles (two exchanges) so that each is left
// with 16 consecutive elements of one sub-row.  (Gathering the nibbles of each sub-row's words over 16 lanes took 110
// vector instructions, this 50.)
__device__ __forceinline__ unsigned sign_half(const float4 (&p)[SUBROWS], int n_valid)
{
    const int lane = lane_id();
    unsigned v = 0;                     // bits 4k .. 4k + 3: this lane's elements of sub-row k
#pragma unroll
    for (int k = SUBROWS - 1; k >= 0; --k) {
        unsigned nib = (p[k].x >= 0.f ? 1u : 0u) | (p[k].y >= 0.f ? 2u : 0u) | (p[k].z >= 0.f ? 4u : 0u) |
                       (p[k].w >= 0.f ? 8u : 0u);
        if (n_valid != TILE) {
            const int left = n_valid - local_base(k);
            nib = left >= 4 ? nib : left > 0 ? nib & ((1u << left) - 1u) : 0u;
        }
        v |= nib << (4 * k);
    }
    // lanes 0 and 1 of a quad keep sub-rows 0 and 1, lanes 2 and 3 the others; then even lanes the first, odd the second
    const unsigned w = row_move<EF_DPP_XOR2>(v);
    const unsigned t = __builtin_amdgcn_perm(w, v, (lane & 2) ? 0x0c0c0105u : 0x0c0c0400u);
    const unsigned u = row_move<EF_DPP_XOR1>(t);
    const unsigned own = (lane & 1) ? 0xf0f0u : 0x0f0fu;
    return (t & own) | (((lane & 1) ? u >> 4 : u << 4) & (own ^ 0xffffu));
}
// Sign bits of a quarter of a tile, stored from word `at` on: the 64 halves of a wavefront fill 128 contiguous bytes.
// WORDS: four lanes' halves are put together first, and lanes 0 to 3 of each row of 16 store 8 bytes, which the momentum
// worker with one workgroup per tile prefers (16 workers, 2734 tiles: 598.1 us against 600.6) and the others do not (server, 16
// workers, 86 000 tiles: 892 against 868; momentum-free worker in blocks of 30 011: 66.6 against 66.0).
template <bool WORDS>
__device__ __forceinline__ void store_quarter_signs(unsigned half, uint64_t *signs, int64_t at, int64_t W)
{
    if constexpr (WORDS) {
        const unsigned lo = half | (row_move<EF_DPP_FROM_4_ON>(half) << 16), hi = row_move<EF_DPP_FROM_8_ON>(lo);
        const int64_t w = at + 4 * (lane_id() & 3) + (lane_id() >> 4);
        if ((lane_id() & 15) < SUBROWS && w < W) signs[w] = ((uint64_t)hi << 32) | (uint64_t)lo;
    } else {
        const int64_t h = 4 * at + 16 * (lane_id() & 3) + (lane_id() >> 2);
        if (h < 4 * W) reinterpret_cast<uint16_t *>(signs)[h] = (uint16_t)half;
    }
}

// Sign words of the tile whose values are in p.
template <bool WORDS>
__device__ __forceinline__ void store_signs(const float4 (&p)[SUBROWS], int n_valid, uint64_t *signs,
                                            int64_t tile_start, int64_t W)
{
    store_quarter_signs<WORDS>(sign_half(p, n_valid), signs, (tile_start >> 6) + wave_id() * 16, W);
}

// fp64 sum of |p| over the thread's valid elements, sub-row by sub-row
__device__ __forceinline__ double abs_sum(const float4 (&p)[SUBROWS], int n_valid)
{
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        const int lb0 = local_base(k);
        const float a[4] = {fabsf(p[k].x), fabsf(p[k].y), fabsf(p[k].z), fabsf(p[k].w)};
        double row = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) row += (n_valid == TILE || lb0 + c < n_valid) ? (double)a[c] : 0.0;
        acc += row;
    }
    return acc;
}

// LDS of a workgroup: what every kernel needs for reductions and broadcasts ...
struct SyncShared {
    double red[2 * NWAVES];     // one a wavefront, two where it has two tiles (server_pair)
    int flag[2];
    unsigned ticket;
    unsigned park[2];           // waits that ran out (head, tail): number of the entry, and PARK_FORMS
    unsigned long long own[2];  // this workgroup's own segments to see to (0: none)
};
// ... and what the kernels that cut a tile into segments need on top of it.
struct TileShared : SyncShared {
    alignas(16) float val[TILE];    // |p| per element, then the element's scale (closed segments)
    double open_sum[2];
    int long_list[MAX_LONG];
    int n_long;
};

// ------------------------------------------------- per-set scratch views ---

__device__ __forceinline__ unsigned long long *set_part(const Scratch &X, const Layout &L, int set)
{
    return X.part + (int64_t)set * 2 * L.ntiles;
}
__device__ __forceinline__ unsigned long long set_tag(const Scratch &X, int set)
{
    return (X.tags >> (set - X.set_base)) & 1ull;
}

// -------------------------------------------------- the end of the call ---

// The call is over: count it, flip the tags of the sets it used, clear the words the next
// call will use (one wavefront).  now: what *state holds.
__device__ __forceinline__ void advance_call(CallState *state, const CallState &now, const Scratch &X, int nsets, int lazy)
{
    const int lane = lane_id();
    if (lane < 4) X.next_cnt[2 * lane] = 0u;
    if (lane <= TAKEN) X.next_cnt[ARRIVE_AT + lane * ARRIVE_STRIDE] = 0u;
    if (lane != 0) return;
    const unsigned long long used = nsets >= 64 ? ~0ull : ((1ull << nsets) - 1ull);
    state->calls = now.calls + 1u;
    if (X.set_base == 0) {
        state->worker_tags = now.worker_tags ^ used;
        // with the deferred correction on, the large blocks of these sets now hold p
        state->worker_pending = lazy ? (now.worker_pending | used) : (now.worker_pending & ~used);
    } else {
        state->server_tag = now.server_tag ^ 1u;
        state->server_pending = lazy ? 1u : 0u;
    }
}

// This call's words of the count (its defer_cnt is the first word of its parity).
__device__ __forceinline__ unsigned *arrive_word(const Scratch &X, unsigned g) { return X.defer_cnt + ARRIVE_AT + g * ARRIVE_STRIDE; }

// Thread 0 counts its workgroup in; the answer goes to arrived().  Every wavefront has read the call state for itself, and the
// last workgroup to be counted changes it: a barrier has to lie between any wavefront's open_call and this, with
// what it loaded in its registers.  (What is behind a barrier that hands over LDS contents is: the wait ahead of one is for
// scalar loads, too.)  Called when the tile's sums are posted: an atomic ahead of
// the loads of scales and block offsets would keep the compiler from making them scalar loads (momentum-free worker, 16 workers,
// 10 606 dense tiles: 1370 -> 1460 us), and where many values are still to come it costs the server's pairs 7
// spilled registers.  (The lane number, 0 here, keeps the compiler from
// making one addition of the wavefront's, whose answer it would wait for at once.)
template <int WAVE = 0>
__device__ __forceinline__ unsigned arrive(const Scratch &X)
{
    unsigned before = 0u;
    if (X.ends && threadIdx.x == 64 * WAVE) {
        unsigned *at = arrive_word(X, blockIdx.x % ARRIVE_GROUPS) + __builtin_amdgcn_mbcnt_lo(~0u, 0u);
        before = __hip_atomic_fetch_add(at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return before;
}
__device__ __forceinline__ unsigned arrive_groups(const ScratchRef &R) { return min((unsigned)R.columns, (unsigned)ARRIVE_GROUPS); }

__device__ __forceinline__ unsigned arrive(const Scratch &X, SyncShared &S)
{
    if (X.ends && threadIdx.x == 0) S.own[0] = S.own[1] = 0ull;
    return arrive(X);
}

// The last workgroup to have counted itself in steps the call state, one wavefront alone.  Returns to that one the number
// of entries that are left, to the last one of a group how many there are so far, 0 to all others: if it is not 0, that
// wavefront is to help with them at its end.  Called when the answer is likely to be there: after the wait for a scale.
template <int WAVE = 0>
__device__ __forceinline__ unsigned arrived(unsigned before, const Scratch &X)
{
    if (!X.ends || uniform_u32(threadIdx.x >> 6) != WAVE) return 0u;
    const ScratchRef &R = call_args().R;
    const unsigned g = blockIdx.x % ARRIVE_GROUPS;
    if (uniform_u32(before) + 1u != (unsigned)R.nsets * (((unsigned)R.columns + ARRIVE_GROUPS - 1u - g) / ARRIVE_GROUPS)) return 0u;
    typedef __attribute__((address_space(4))) const void *Segment;
    Segment state = (Segment)R.step;        // nobody has changed it yet: a scalar load, like the first one
    asm("" : "+s"(state));
    const CallState now = *(const CallState *)state;
    unsigned top = 0u;
    if (lane_id() == 0) top = atomicAdd(arrive_word(X, ARRIVE_GROUPS), 1u);
    top = uniform_u32(top);
    if ((top & ARRIVED_MASK) + 1u != arrive_groups(R)) return top / PARKED_ONE;
    if (lane_id() == 0) __hip_atomic_store(arrive_word(X, LEFT), top / PARKED_ONE + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    advance_call(R.step, now, X, R.nsets, R.lazy);
    return top / PARKED_ONE;
}

// Thread 0: a wait has run out.  If all workgroups have begun, this one sees to the segment itself at its end, where the sums
// are sure to come; else the segment gets the number of an entry.
__device__ __forceinline__ void give_up(const Scratch &X, unsigned *park, unsigned forms)
{
    const unsigned top = atomicAdd(arrive_word(X, ARRIVE_GROUPS), PARKED_ONE);
    *park = ((top & ARRIVED_MASK) == arrive_groups(call_args().R) ? PARK_OWN : top / PARKED_ONE) | forms;
}
// What the workgroup has stored, and its wavefronts have waited for, is there for all others to see.  One wavefront.  The second wait is the
// write-back's: the fence's own is dropped by the compiler where it knows of no store on its way, and does not count that.
__device__ __forceinline__ void release_stores()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __builtin_amdgcn_s_waitcnt(0);
}
// And the segment has been stored as p: an entry, in ScratchRef::parked or the workgroup's own.  One thread, after a release.
__device__ __forceinline__ void leave_entry(unsigned park, unsigned long long both, const Scratch &X, int set, int32_t tile, int which,
                                            unsigned long long *own)
{
    const unsigned long long entry = parked_entry(X.epoch, set, tile, which, both | ((park & PARK_FORMS) ? PARKED_FORMS : 0ull));
    if ((park & ~PARK_FORMS) == PARK_OWN)
        *own = entry;
    else
        __hip_atomic_store(call_args().R.parked + (park & ~PARK_FORMS), entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------ cross-tile block reductions ---

struct BlockSpan {
    int64_t bs, be;             // element range
    int64_t t0;                 // first tile
    int n;                      // tiles
};

__device__ __forceinline__ BlockSpan span_of(int64_t bs, int64_t be)
{
    BlockSpan s;
    s.bs = bs;
    s.be = be;
    s.t0 = bs / TILE;
    s.n = (int)((be - 1) / TILE - s.t0 + 1);
    return s;
}
__device__ __forceinline__ BlockSpan block_span(const Layout &L, int64_t b) { return span_of(L.offs[b], L.offs[b + 1]); }

// Does the block own a whole tile?  Its first tile is shared (or ragged) if it
// starts inside it, its last tile if it ends inside it; the tiles between are
// its own.
__device__ __forceinline__ bool has_uniform_tile(const BlockSpan &s)
{
    return s.n - ((s.bs % TILE) != 0 ? 1 : 0) - ((s.be % TILE) != 0 ? 1 : 0) >= 1;
}

// One-pass blocks: their scale is formed and posted inside the main kernel(s) of the call.
__device__ __forceinline__ bool is_counted(const Layout &L, const BlockSpan &s)
{
    return s.n >= 2 && s.n <= L.fuse_limit;
}

// A one-pass block without a whole tile: all its tiles are mixed ones, which form its scale (in
// the block's last tile) and finish its segments among themselves.
__device__ __forceinline__ bool finishes_with_mixed(const Layout &L, const BlockSpan &s)
{
    return is_counted(L, s) && !has_uniform_tile(s);
}

// A block larger than fuse_limit: its whole tiles from this one on keep p and wait for the scale like those of a one-pass
// block do, so that the pass over what was parked leaves them out; its last whole tile forms the scale.  As many as are sure to be resident are kept, the limit again.  us without
// and with: server, 16 workers, a block of 12 565 tiles in 86 000, 901 / 876 (the pass over what is parked 68 -> 59, and
// k_tail no longer adds up 12 565 partial sums, 24 -> 5); worker, the same layout, 1301 / 1289; step of 4 workers with
// four blocks of 2049 tiles on the server, 917 / 905, and 891 with pairs, whose limit is 1792.
__device__ __forceinline__ int64_t first_kept(const Layout &L, const BlockSpan &s)
{
    const int first = (s.bs % TILE) != 0 ? 1 : 0, whole = s.n - first - ((s.be % TILE) != 0 ? 1 : 0);
    return first_kept(s.t0 + first, whole, L.keep);
}

// Scratch word of block b's segment in tile t: slot 1 of the block's first tile
// if b starts inside that tile (it is then the tile's last segment), slot 0
// everywhere else (first or only segment).
__device__ __forceinline__ int64_t part_index(int64_t t, const BlockSpan &s)
{
    return 2 * t + ((t == s.t0 && (s.bs % TILE) != 0) ? 1 : 0);
}

// The block's last whole tile (meaningful if it has one).
__device__ __forceinline__ int64_t last_whole_tile(const BlockSpan &s)
{
    return s.t0 + s.n - 1 - ((s.be % TILE) != 0 ? 1 : 0);
}

// The tile whose workgroup forms the block's scale: the block's last whole tile, or its last tile
// if it has no whole one.
__device__ __forceinline__ int64_t gatherer_tile(const Layout &L, const BlockSpan &s)
{
    return has_uniform_tile(s) ? last_whole_tile(s) : s.t0 + s.n - 1;
}

// The ready word of a block that spans tiles: where its scale is posted with the call number and
// the workgroups of its other tiles look for it.  Every block has a 128-byte line of its own, found
// through its gatherer tile (different blocks have different gatherer tiles): with the words of
// neighbouring blocks in one line, the gatherers' stores and the other tiles' polls of up to 16
// blocks met in that line, which cost the kernels that wait in place up to a third of their
// time on blocks of 16 to 64 tiles (worker 9.0 -> 6.7 ms, server 0.81 -> 0.44 ms on 2^28 elements
// in blocks of 2^16) and a few percent on blocks of 256 tiles.
constexpr int READY_STRIDE = 16;    // 64-bit words
__device__ __forceinline__ unsigned long long *ready_word(const Scratch &X, const Layout &L, int set, const BlockSpan &sp)
{
    return X.ready + ((int64_t)set * L.ntiles + gatherer_tile(L, sp)) * READY_STRIDE;
}

// What a uniform tile has to follow up on after posting its partial: the block
// whose scale it must form (it is that block's last whole tile), or -1.
struct Posted {
    int gather;
    BlockSpan sp;               // of that block
};

__device__ __forceinline__ void clear_posted(Posted &P) { P.gather = -1; }

// Post the partial sum of an open segment.  which: 0 = the tile's first (or
// only) segment, 1 = its last segment.  Never waits.
__device__ __forceinline__ void store_partial(double partial, int which, int32_t tile, const Layout &L,
                                              const Scratch &X, int set)
{
    if (threadIdx.x == 0) {
        const unsigned long long w =
            (unsigned long long)__double_as_longlong(partial) | (set_tag(X, set) ? TAG_BIT : 0ull);
        __hip_atomic_store(set_part(X, L, set) + 2 * (int64_t)tile + which, w, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Sum of block b's partials once the kernel that posted them has finished.
// Same order as gather_scale.  Called by every thread of the workgroup.
__device__ __forceinline__ double sum_block_partials(const Layout &L, int64_t b, const unsigned long long *part,
                                                     double *red)
{
    const BlockSpan sp = block_span(L, b);
    double acc = 0.0;
    // eight words in flight a thread: a block of 12 565 tiles is 49 of them, one after the other 25 us
    for (int64_t i0 = threadIdx.x; i0 < sp.n; i0 += 8 * THREADS) {
        unsigned long long w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = i0 + q * THREADS;
            w[q] = i < sp.n ? part[part_index(sp.t0 + i, sp)] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += __longlong_as_double((long long)(w[q] & ~TAG_BIT));
    }
    return block_sum(acc, red);
}

// Wait (bounded) until every tile of block b has posted this call's partial,
// then form the block's scale.  Called by every thread of the workgroup with
// the same arguments; returns the same answer to all of them.
constexpr int GATHER_DEEP = 4;      // partial words a thread has in flight

__device__ __forceinline__ bool gather_scale(const BlockSpan &sp, const Layout &L, const Scratch &X, int set, int spin_limit,
                                             SyncShared &S, float *s)
{
    const unsigned long long *part = set_part(X, L, set);
    const unsigned long long tag = set_tag(X, set);
    // Thread t is in charge of tiles t, t + 256, ..., and adds them in this order (that of sum_block_partials), a few at a
    // time: all of them are asked for in every round, so that the loads of a round overlap, until all have this
    // call's tag.  Only rounds that found a word missing count as polls (a chunk takes its last one back): a block may have
    // any number of tiles.  Counted where the words are found missing, a bottleneck network's server call is 0.3 of 20.2 us
    // slower; with a budget for each chunk, sixteen workers' is 30 of 870.
    double acc = 0.0;
    int polls = 0, ok = 1;
#pragma unroll 1
    for (int from = 0; from < sp.n && ok; from += GATHER_DEEP * THREADS, --polls) {
        unsigned long long w[GATHER_DEEP];
        const int mine = from + (int)threadIdx.x;
#pragma unroll
        for (int q = 0; q < GATHER_DEEP; ++q) w[q] = tag << 63;         // past the block: +0 with this call's tag
        for (;;) {
            if (polls++ >= spin_limit) {
                ok = 0;
                break;
            }
#pragma unroll
            for (int q = 0; q < GATHER_DEEP; ++q)
                if (mine + q * THREADS < sp.n)
                    w[q] = __hip_atomic_load(part + part_index(sp.t0 + mine + q * THREADS, sp), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
            bool all = true;
#pragma unroll
            for (int q = 0; q < GATHER_DEEP; ++q) all = all && (w[q] >> 63) == tag;
            if (all) break;
            __builtin_amdgcn_s_sleep(8);
        }
#pragma unroll
        for (int q = 0; q < GATHER_DEEP; ++q) acc += __longlong_as_double((long long)(w[q] & ~TAG_BIT));
    }
    if (!__syncthreads_and(ok)) return false;
    const double total = block_sum(acc, S.red);
    *s = (float)(total / (double)(sp.be - sp.bs));
    return true;
}

// A scale is there: written out and posted for the block's other tiles.  One thread.
__device__ __forceinline__ void post_scale(int64_t b, const BlockSpan &sp, float s, const Layout &L, const Scratch &X, int set,
                                           float *scales_out)
{
    scales_out[b] = s;
    __hip_atomic_store(ready_word(X, L, set, sp), ((unsigned long long)X.epoch << 32) | (unsigned long long)__float_as_uint(s),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroup that holds the gatherer tile of one-pass block b forms the
// scale from the partials (waiting, bounded, for those still in flight: every
// other tile of the block was handed out earlier), writes it out and posts it
// for the block's other tiles.  Called by every thread of that workgroup;
// returns to all of them whether the scale could be formed, and the scale.
__device__ __forceinline__ bool finish_block(int64_t b, const BlockSpan &sp, const Layout &L, const Scratch &X, int set,
                                             float *scales_out, SyncShared &S, int slot, float *scale)
{
    float s = 0.f;
    const bool ok = gather_scale(sp, L, X, set, X.spin_limit, S, &s);
    if (threadIdx.x == 0) {
        if (ok) {
            post_scale(b, sp, s, L, X, set, scales_out);
        } else {
            const unsigned k = atomicAdd(X.fin_cnt, 1u);
            if (X.ends) {
                give_up(X, &S.park[slot], PARK_FORMS);
            } else {
                X.fin_list[k] = ((unsigned long long)set << 32) | (unsigned long long)b;
            }
        }
    }
    *scale = s;
    return ok;
}

// Follow up on what a uniform tile posted: if it is its block's last whole
// tile, finish that block.  Called by every thread of the workgroup.
__device__ __forceinline__ void resolve_posted(const Posted &P, const Layout &L, const Scratch &X, int set,
                                               float *scales_out, SyncShared &S)
{
    float s;
    if (P.gather >= 0) (void)finish_block(P.gather, P.sp, L, X, set, scales_out, S, 0, &s);
}

// Thread 0's early look at the ready word of block b (b < 0: none).
__device__ __forceinline__ unsigned long long peek_ready(int b, const Layout &L, const Scratch &X, int set)
{
    unsigned long long w = 0ull;           // epoch 0 is never used
    if (threadIdx.x == 0 && b >= 0)
        w = __hip_atomic_load(ready_word(X, L, set, block_span(L, b)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return w;
}

// Wait (bounded) until the block's gatherer has posted its scale of this call.
// `peeked` is thread 0's earlier look at the word (see peek_ready).  Called by
// every thread of the workgroup; same answer to all of them.
__device__ __forceinline__ bool wait_ready_at(const unsigned long long *word, unsigned long long peeked, const Scratch &X,
                                              SyncShared &S, float *s)
{
    if (threadIdx.x == 0) {
        unsigned long long w = peeked;
        int found = ((unsigned)(w >> 32) == X.epoch) ? 1 : 0;
        for (int it = 0; !found && it < X.spin_limit; ++it) {
            w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            found = ((unsigned)(w >> 32) == X.epoch) ? 1 : 0;
            if (!found) __builtin_amdgcn_s_sleep(8);
        }
        if (X.spin_limit <= 0) found = 0;   // a zero budget means: never take the one-pass route
        S.flag[0] = found;
        S.flag[1] = (int)(unsigned)w;
    }
    __syncthreads();
    const bool ok = S.flag[0] != 0;
    *s = __uint_as_float((unsigned)S.flag[1]);
    __syncthreads();
    return ok;
}

__device__ __forceinline__ bool wait_ready(const BlockSpan &sp, unsigned long long peeked, const Layout &L, const Scratch &X,
                                           int set, SyncShared &S, float *s)
{
    return wait_ready_at(ready_word(X, L, set, sp), peeked, X, S, s);
}

// Leave a segment whose p gets parked in the residual buffer to the kernels
// that run after this one.
__device__ __forceinline__ void defer_segment(int32_t tile, int which, const Scratch &X, int set)
{
    if (threadIdx.x == 0) {
        const unsigned i = atomicAdd(X.defer_cnt, 1u);
        X.defer_list[i] = ((unsigned long long)set << 33) | ((unsigned long long)tile << 1) | (unsigned)which;
    }
}

// The scale of a one-pass block (or one with kept tiles), which the gatherer (`forms`) makes of the partial sums, writes out
// and posts, and the others wait for; both bounded.  False: the wait ran out, and p is to be parked (park_segment).  Called by
// every thread of the workgroup; same answer to all of them.  word: the block's ready word.
__device__ __forceinline__ bool wait_scale(const unsigned long long *word, const Scratch &X, SyncShared &S, int slot, float *scale)
{
    if (wait_ready_at(word, 0ull, X, S, scale)) return true;
    if (X.ends && threadIdx.x == 0) give_up(X, &S.park[slot], 0u);
    return false;
}
__device__ __forceinline__ bool block_scale(bool forms, int64_t b, const BlockSpan &sp, const Layout &L, const Scratch &X, int set,
                                            float *scales_out, SyncShared &S, int slot, float *scale)
{
    if (!forms) return wait_scale(ready_word(X, L, set, sp), X, S, slot, scale);
    return finish_block(b, sp, L, X, set, scales_out, S, slot, scale);
}

// The segment (both: the whole tile and the next one) whose wait ran out has been stored as p: an entry for whoever ends
// the call.  One wavefront releases for all of them, whose stores have reached the L2 by then.
__device__ __forceinline__ void park_segment(int32_t tile, int which, bool both, const Scratch &X, int set, SyncShared &S)
{
    if (!X.ends) {
        defer_segment(tile, which, X, set);
        if (both) defer_segment(tile + 1, which, X, set);
        return;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(X.defer_cnt, both ? 2u : 1u);
        release_stores();
        leave_entry(S.park[which], both ? PARKED_BOTH : 0ull, X, set, tile, which, &S.own[which]);
    }
    __syncthreads();
}

// ------------------------------------------------------- tile compression ---

// A thread's elements among the segments of a mixed tile, sub-row by sub-row: bits 0-3: a segment starts at
// element c; above: segments started before element 0 (so the segment in progress there, plus one).
struct TilePlace {
    unsigned row[SUBROWS];
    __device__ __forceinline__ unsigned starts(int k) const { return row[k] & 15u; }
    __device__ __forceinline__ int seg(int k) const { return (int)(row[k] >> 4) - 1; }
};
__device__ __forceinline__ TilePlace tile_place(const StartWord *words, const TileRec &T)
{
    TilePlace q;
    const unsigned sh = (threadIdx.x & 7u) * 4u;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        const StartWord w = words[(int64_t)T.words * TILE_WORDS + (local_base(k) >> 5)];
        q.row[k] = ((w.starts >> sh) & 15u) | ((w.rank + (unsigned)__popc(w.starts & ((1u << sh) - 1u))) << 4);
    }
    return q;
}
// Mixed tile of any number of segments, among the dense ones or ahead of the persistent kernel: sign
// words; segmented fp64 sums through LDS; scales and residuals e' = p - Delta of the
// closed segments; partial sums of the (at most two) open segments posted, and
// their residuals finished too where the block's scale forms inside this kernel
// (bounded waits), else their elements stored as p for the kernel that ends the
// call.  (Section 3.2 and e_{t+1} = p_t - Delta_t of Algorithm 4.)  The sums are those of
// segment_sum, short segments a thread each.
// Returns what arrived() answers.
__device__ __forceinline__ unsigned compress_mixed(float4 (&p)[SUBROWS], const Layout &L, const TileRec &T, int32_t tile, int n_valid,
                                                   uint64_t *signs, float *scales_out, float *err_tile,
                                                   const Scratch &X, int set, TileShared &S)
{
    const int64_t tile_start = (int64_t)tile * TILE;
    const int32_t fb = T.fb, lb = T.fb + abs(T.nseg) - 1;
    store_signs<false>(p, n_valid, signs, tile_start, L.W);

    const int nseg = lb - fb + 1;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        float4 a = make_float4(fabsf(p[k].x), fabsf(p[k].y), fabsf(p[k].z), fabsf(p[k].w));
        *reinterpret_cast<float4 *>(&S.val[local_base(k)]) = a;
    }
    if (threadIdx.x == 0) S.n_long = 0;
    __syncthreads();
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
        double acc = 0.0;               // most are a few elements: ordered_sum's groups of eight cost more than they hide
        for (int j = lo; j < hi; ++j) acc += (double)S.val[j];
        const bool open = (sg == 0 && head_open) || (sg == nseg - 1 && tail_open);
        if (open) {
            S.open_sum[sg == 0 ? 0 : 1] = acc;
        } else {
            const float sc = (float)(acc / (double)(be - bs));
            scales_out[b] = sc;
            for (int j = lo; j < hi; ++j) S.val[j] = sc;
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
        const double acc = wave_sum(ordered_sum<64>(S.val, lo + lane_id(), hi, 0.0));
        const bool open = (sg == 0 && head_open) || (sg == nseg - 1 && tail_open);
        if (open) {
            if (lane_id() == 0) S.open_sum[sg == 0 ? 0 : 1] = acc;
        } else {
            const float sc = (float)(acc / (double)(be - bs));
            if (lane_id() == 0) scales_out[b] = sc;
            for (int j = lo + lane_id(); j < hi; j += 64) S.val[j] = sc;
        }
    }
    __syncthreads();
    const int head_end = head_open ? (int)min(L.offs[fb + 1] - tile_start, (int64_t)n_valid) : 0;
    const int tail_begin = tail_open ? (int)(L.offs[lb] - tile_start) : TILE;
    if (head_open) store_partial(S.open_sum[0], 0, tile, L, X, set);
    if (tail_open) store_partial(S.open_sum[1], 1, tile, L, X, set);
    const unsigned before = arrive(X, S);
    // An open segment whose block has no whole tile is finished in place: all tiles of such a
    // block are mixed ones, handed out before any whole tile and in ascending order.  The first
    // segment's block ends in this tile, which makes this workgroup the one that forms its scale;
    // the last segment's block goes on, and its scale comes from the next mixed tile.  The segments
    // of other blocks, and any whose wait runs out, keep p in the residual buffer for the kernel
    // that ends the call.
    float s_head = 0.f, s_tail = 0.f;
    bool fin_head = false, fin_tail = false;
    bool park_head = false, park_tail = false;
    if (head_open && finishes_with_mixed(L, block_span(L, fb))) {
        fin_head = finish_block(fb, block_span(L, fb), L, X, set, scales_out, S, 0, &s_head);
        park_head = !fin_head;
    }
    if (tail_open && finishes_with_mixed(L, block_span(L, lb))) {
        fin_tail = wait_scale(ready_word(X, L, set, block_span(L, lb)), X, S, 1, &s_tail);
        park_tail = !fin_tail;
    }
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) {
        const int lb0 = local_base(k);
        const float4 sc = *reinterpret_cast<const float4 *>(&S.val[lb0]);
        const float pv[4] = {p[k].x, p[k].y, p[k].z, p[k].w};
        const float sv[4] = {sc.x, sc.y, sc.z, sc.w};
        float ev[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = lb0 + c;
            if (j < head_end)
                ev[c] = fin_head ? residual(pv[c], s_head) : pv[c];
            else if (j >= tail_begin)
                ev[c] = fin_tail ? residual(pv[c], s_tail) : pv[c];
            else
                ev[c] = residual(pv[c], sv[c]);
        }
        p[k] = make_float4(ev[0], ev[1], ev[2], ev[3]);
    }
    store_tile(err_tile, p, n_valid);
    if (park_head) park_segment(tile, 0, false, X, set, S);
    if (park_tail) park_segment(tile, 1, false, X, set, S);
    __syncthreads();            // S.val is free again
    return arrived(before, X);
}

// Deferred correction of a uniform tile's residual as loaded (see Scratch::lazy_scales): if the
// tile's block is larger than fuse_limit and the set's last call left p in the buffer, what that
// call's payload stood for is subtracted.  The scale is looked up before the tile's loads are
// issued (two dependent scalar loads that then overlap with them) and applied once they are in.
// Called by every thread with the same block and set.
struct LoadedCorrection {
    float s;
    bool on;
};
__device__ __forceinline__ LoadedCorrection loaded_correction(const Layout &L, int32_t b, const Scratch &X, int set)
{
    LoadedCorrection c;
    c.s = 0.f;
    c.on = false;
    if (!L.lazy || !((X.pending >> (set - X.set_base)) & 1ull)) return c;
    const int32_t li = L.late_index[b];
    if (li < 0) return c;
    c.s = X.lazy_scales[(int64_t)set * X.lazy_stride + li];
    c.on = true;
    return c;
}
__device__ __forceinline__ void correct_loaded_residual(float4 (&e)[SUBROWS], const LoadedCorrection &c)
{
    if (!c.on) return;
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k) residual4(e[k], c.s);
}

// Uniform tile (inside one block b): sign words and the tile's fp64 sum.
// Returns what is left to do with it:
//   UNI_DONE    the block is this tile alone: scale and residual written;
//   UNI_PARKED  block larger than fuse_limit: partial posted, p parked for the
//               kernel that ends the call (P may say that this tile must form the scale all the same);
//   UNI_PENDING partial posted: p stays with the caller until the block's
//               scale is posted; P says whether this tile must form it.
//   UNI_HELD    (only with hold = true) as UNI_PARKED, but p is still to be written by the caller,
//               after sync_group_wait.
enum { UNI_DONE = 0, UNI_PARKED = 1, UNI_PENDING = 2, UNI_HELD = 3 };

template <bool WORDS = false>
__device__ __forceinline__ int compress_uniform(float4 (&p)[SUBROWS], const Layout &L, int32_t tile, int32_t b,
                                                const BlockSpan &sp, int n_valid, uint64_t *signs, float *scales_out,
                                                float *err_tile, const Scratch &X, int set, SyncShared &S, Posted &P,
                                                bool hold = false)
{
    const int64_t tile_start = (int64_t)tile * TILE;
    clear_posted(P);
    store_signs<WORDS>(p, n_valid, signs, tile_start, L.W);
    const double total = block_sum(abs_sum(p, n_valid), S.red);
    if (sp.bs >= tile_start && sp.be <= tile_start + TILE) {
        const float s = (float)(total / (double)(sp.be - sp.bs));
        if (threadIdx.x == 0) scales_out[b] = s;
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) residual4(p[k], s);
        store_tile(err_tile, p, n_valid);
        return UNI_DONE;
    }
    store_partial(total, 0, tile, L, X, set);
    const bool counted = is_counted(L, sp);
    if ((counted || L.keep > 0) && (int64_t)tile == gatherer_tile(L, sp)) {
        P.gather = b;
        P.sp = sp;
    }
    if (counted || (L.keep > 0 && (int64_t)tile >= first_kept(L, sp))) return UNI_PENDING;
    if (hold && L.sync_group > 1) return UNI_HELD;
    store_tile(err_tile, p, n_valid);
    return UNI_PARKED;
}

// Write the residual of a uniform tile of counted block b whose p was kept
// (e_{t+1} = p_t - Delta_t, Algorithm 4), waiting (bounded) for the scale; if
// the wait runs out, p is parked and the segment deferred.
__device__ __forceinline__ void finish_uniform(float4 (&p)[SUBROWS], int32_t tile, int n_valid, const BlockSpan &sp,
                                               unsigned long long peeked, float *err_tile, const Layout &L,
                                               const Scratch &X, int set, SyncShared &S, bool may_wait = true)
{
    float s = 0.f;
    const bool ok = may_wait && wait_ready(sp, peeked, L, X, set, S, &s);
    if (ok) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) residual4(p[k], s);
    } else {
        defer_segment(tile, 0, X, set);
    }
    store_tile(err_tile, p, n_valid);
}

// A tile where at most FEW_SEGS blocks meet, or the ragged end of the vector, taken among the whole tiles: the
// ends of large blocks with the small ones between them (weights, then biases and norms), which is what
// the mixed tiles of a network's layout are.  The segments are summed from LDS, a wavefront each, and
// corrected in the registers the whole tiles need anyway, every thread's elements masked by the segment's range;
// an open segment waits for its block's scale like a whole tile does.  (Mixed tiles at the head of the
// grid, with the segment code for any number of segments, cost the kernel registers, its first
// workgroups 20 us, and the segments of blocks with whole tiles a pass of their own in the kernel that
// ends the call: 25 M elements in blocks of 64 tiles and 7 elements, server call with 7 workers 65 us
// against 48 for blocks of 64 tiles; 53 now.  Momentum-free worker in blocks of 30 011: 88 -> 66 us.)
// bound[i]: local index of the end of segment i-1 = start of segment i, in LDS.
struct FewShared {
    int bound[FEW_SEGS + 1];
    float scale[FEW_SEGS];      // of the segments; 0 leaves p as it is
    double sum[FEW_SEGS];
};
// Called by the whole workgroup early; a barrier comes before the first use.
__device__ __forceinline__ void few_bounds(const Layout &L, const TileRec &T, int64_t tile_start, int n_valid, int *bound)
{
    if ((int)threadIdx.x <= T.nseg) {
        const int64_t at = L.offs[T.fb + (int)threadIdx.x] - tile_start;
        bound[threadIdx.x] = (int)min(max(at, (int64_t)0), (int64_t)n_valid);
    }
}
__device__ __forceinline__ int few_bound(const int *bound, int i) { return (int)uniform_u32((unsigned)bound[i]); }
// Does this wavefront's sub-row k have elements of [lo, hi)?  Most segments touch one or two of a tile's 16.
__device__ __forceinline__ bool few_touches(int k, int lo, int hi)
{
    const int first = (int)uniform_u32(threadIdx.x >> 6) * 1024 + k * 256;
    return first < hi && first + 256 > lo;
}
// val: TILE floats of LDS.
// Returns what arrived() answers.
template <bool WORDS = false>
__device__ __forceinline__ unsigned compress_few(float4 (&p)[SUBROWS], const Layout &L, const TileRec &T, int32_t tile, int n_valid,
                                                 uint64_t *signs, float *scales_out, float *err_tile, const Scratch &X, int set,
                                                 SyncShared &S, FewShared &F, float *val)
{
    const int64_t tile_start = (int64_t)tile * TILE;
    const int nseg = T.nseg;
    const BlockSpan hs = span_of(T.bs(), T.be());
    const bool head_open = hs.bs < tile_start || hs.be > tile_start + TILE, tail_open = T.tail != 0;
    store_signs<WORDS>(p, n_valid, signs, tile_start, L.W);
#pragma unroll
    for (int k = 0; k < SUBROWS; ++k)
        *reinterpret_cast<float4 *>(val + local_base(k)) = make_float4(fabsf(p[k].x), fabsf(p[k].y), fabsf(p[k].z), fabsf(p[k].w));
    __syncthreads();                // that, and the bounds
#pragma unroll 1
    for (int sg = (int)uniform_u32(threadIdx.x >> 6); sg < nseg; sg += NWAVES) {
        const double total = segment_sum(val, few_bound(F.bound, sg), few_bound(F.bound, sg + 1));
        if (lane_id() == 0) F.sum[sg] = total;
    }
    __syncthreads();
    // what others may wait for goes out first
    if (head_open) store_partial(F.sum[0], 0, tile, L, X, set);
    if (tail_open) store_partial(F.sum[nseg - 1], 1, tile, L, X, set);
    const unsigned before = arrive(X, S);
    if ((int)threadIdx.x < nseg) {
        const int sg = (int)threadIdx.x;
        if (!(sg == 0 && head_open) && !(sg == nseg - 1 && tail_open)) {
            const float s = (float)(F.sum[sg] / (double)(F.bound[sg + 1] - F.bound[sg]));
            scales_out[T.fb + sg] = s;
            F.scale[sg] = s;
        }
    }
    bool park_head = false, park_tail = false;
    if (head_open) {
        float s = 0.f;
        if (is_counted(L, hs)) {
            park_head = !block_scale((int64_t)tile == gatherer_tile(L, hs), T.fb, hs, L, X, set, scales_out, S, 0, &s);
            if (park_head) s = 0.f;
        }
        if (threadIdx.x == 0) F.scale[0] = s;
    }
    if (tail_open) {
        float s = 0.f;
        const int n = T.tail >> 1, whole = n - 1 - (T.tail & 1);
        if (n <= L.fuse_limit) {
            // the block starts in this tile: its whole tiles, if any, are the ones between this and its last
            const int64_t gatherer = (int64_t)tile + (whole > 0 ? whole : n - 1);
            park_tail = !wait_scale(X.ready + ((int64_t)set * L.ntiles + gatherer) * READY_STRIDE, X, S, 1, &s);
            if (park_tail) s = 0.f;
        }
        if (threadIdx.x == 0) F.scale[nseg - 1] = s;
    }
    __syncthreads();
#pragma unroll 1
    for (int sg = 0; sg < nseg; ++sg) {
        const int lo = few_bound(F.bound, sg), hi = few_bound(F.bound, sg + 1);
        const unsigned n = (unsigned)(hi - lo);
        const float s = F.scale[sg];
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) {
            if (!few_touches(k, lo, hi)) continue;
            const int j = local_base(k) - lo;
            p[k].x = (unsigned)(j + 0) < n ? residual(p[k].x, s) : p[k].x;
            p[k].y = (unsigned)(j + 1) < n ? residual(p[k].y, s) : p[k].y;
            p[k].z = (unsigned)(j + 2) < n ? residual(p[k].z, s) : p[k].z;
            p[k].w = (unsigned)(j + 3) < n ? residual(p[k].w, s) : p[k].w;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    store_tile(err_tile, p, n_valid);
    if (park_head) park_segment(tile, 0, false, X, set, S);
    if (park_tail) park_segment(tile, 1, false, X, set, S);
    return arrived(before, X);
}

// Writing the residual out in step.  Measured on this machine: workgroups that take consecutive
// tiles and hold their residual tile back until all of them have posted their partial sums (as
// the tiles of a small one-pass block do, which wait for one scale) stream faster than workgroups
// that each write as soon as they are done (2^28 elements, 8 workers: 6.6 ms in blocks of 8 to
// 16 tiles against 7.7 ms without any wait; the momentum tile is written at once in both cases,
// holding it back as well was measured slower).  For a uniform tile of a block larger than
// fuse_limit that is parked nothing has to be waited for, so the kernel that runs one workgroup per tile makes
// it wait for its neighbours instead: the parked tiles of the block form groups of L.sync_group
// consecutive tiles (group_first, group_last); the last tile of a group looks for this call's tag on the partial words of
// the others (posted just before) and then posts the call number in its own ready line, where
// the others look for it.  Both waits are bounded, and nothing depends on their outcome:
// whoever runs out of patience just writes, and is counted.  (Groups cut from all whole tiles could end in a kept one, which
// never comes here: the others then polled until spin_limit, 0.65 ms a call.  Eight blocks of 5 M elements, one
// worker: 851 -> 151 us; 124 M in 12 transformer layers and an embedding: 993 -> 388.)
// Called by every thread of the workgroup, after compress_uniform returned UNI_HELD.
__device__ __forceinline__ void sync_group_wait(int32_t tile, const BlockSpan &sp, const Layout &L, const Scratch &X, int set,
                                                SyncShared &S)
{
    const int64_t g0 = group_first(tile, sp.t0 + ((sp.bs % TILE) != 0 ? 1 : 0), L.sync_group);
    const int64_t g1 = group_last(g0, L.sync_group, first_kept(L, sp));
    if (g1 == g0) return;
    bool lost = X.spin_limit > 0;       // until the wait is over
    // the second word of the tile's line: the first may be the block's ready word
    unsigned long long *line = X.ready + ((int64_t)set * L.ntiles + g1) * READY_STRIDE + 1;
    if ((int64_t)tile == g1) {
        const unsigned long long *part = set_part(X, L, set);
        const unsigned long long tag = set_tag(X, set);
        const int others = (int)(g1 - g0);
        for (int it = 0; it < X.spin_limit; ++it) {
            int all = 1;
            if ((int)threadIdx.x < others) {
                const unsigned long long w = __hip_atomic_load(part + 2 * (g0 + threadIdx.x), __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                all = (w >> 63) == tag ? 1 : 0;
            }
            if (__syncthreads_and(all)) {
                lost = false;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        if (threadIdx.x == 0)
            __hip_atomic_store(line, (unsigned long long)X.epoch << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        if (threadIdx.x == 0) {
            for (int it = 0; it < X.spin_limit; ++it) {
                const unsigned long long w = __hip_atomic_load(line, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((unsigned)(w >> 32) == X.epoch) {
                    lost = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && lost) atomicAdd(X.lost_cnt, 1u);
}

// What the kernels with one workgroup per tile do with a uniform tile once its sum is posted (compress_uniform's answers):
// its block's scale, formed here or waited for in place, then its residual.
// Returns what arrived() answers.
__device__ __forceinline__ unsigned settle_uniform(float4 (&p)[SUBROWS], int kind, const Posted &P, int32_t tile, int32_t b,
                                                   const BlockSpan &sp, float *scales_out, float *err_tile, const Layout &L,
                                                   const Scratch &X, int set, SyncShared &S)
{
    const unsigned before = arrive(X, S);
    float s = 0.f;
    bool ok = false;
    if (kind == UNI_PENDING || P.gather >= 0) ok = block_scale(P.gather >= 0, b, sp, L, X, set, scales_out, S, 0, &s);
    const unsigned left = arrived(before, X);
    if (kind == UNI_HELD) {
        sync_group_wait(tile, sp, L, X, set, S);
        store_tile(err_tile, p, TILE);
    }
    if (kind != UNI_PENDING) return left;
    if (ok) {
#pragma unroll
        for (int k = 0; k < SUBROWS; ++k) residual4(p[k], s);
    }
    store_tile(err_tile, p, TILE);
    if (!ok) park_segment(tile, 0, false, X, set, S);
    return left;
}

// Fill the first half of S.val (read as 16-bit integers) with the segment index of every element of a
// mixed tile (0 past the end of the vector), so that element j can look up scale[fb + seg].
__device__ __forceinline__ void build_segment_index(const Layout &L, int32_t tile, int n_valid, int32_t fb,
                                                    int nseg, TileShared &S)
{
    const int64_t tile_start = (int64_t)tile * TILE;
    uint16_t *seg = reinterpret_cast<uint16_t *>(S.val);
    if (threadIdx.x == 0) S.n_long = 0;
    __syncthreads();
    for (int j = n_valid + (int)threadIdx.x; j < TILE; j += THREADS) seg[j] = 0;
    for (int sg = threadIdx.x; sg < nseg; sg += THREADS) {
        const int lo = (int)max(L.offs[fb + sg] - tile_start, (int64_t)0);
        const int hi = (int)min(L.offs[fb + sg + 1] - tile_start, (int64_t)n_valid);
        if (hi - lo > SMALL_SEG) {
            S.long_list[atomicAdd(&S.n_long, 1)] = sg;
            continue;
        }
        for (int j = lo; j < hi; ++j) seg[j] = (uint16_t)sg;
    }
    __syncthreads();
    const int n_long = S.n_long;
    for (int q = wave_id(); q < n_long; q += NWAVES) {
        const int sg = S.long_list[q];
        const int lo = (int)max(L.offs[fb + sg] - tile_start, (int64_t)0);
        const int hi = (int)min(L.offs[fb + sg + 1] - tile_start, (int64_t)n_valid);
        for (int j = lo + lane_id(); j < hi; j += 64) seg[j] = (uint16_t)sg;
    }
    __syncthreads();
}

// Tile records in another order (plan creation: a list of 4-byte numbers is copied to the device, not 32-byte records).  The
// top bit of a number: the tile and the next one as a pair.
constexpr uint32_t PAIR_BIT = 1u << 31;
__global__ __launch_bounds__(THREADS) void k_take_records(const TileRec *tiles, const uint32_t *order, int n, TileRec *out)
{
    const int i = blockIdx.x * THREADS + threadIdx.x;
    if (i >= n) return;
    TileRec r = tiles[order[i] & ~PAIR_BIT];
    if (order[i] & PAIR_BIT) r.words = TILE_PAIR;
    out[i] = r;
}

// Start words of the mixed tiles (plan creation).  One workgroup per mixed tile.
__global__ __launch_bounds__(THREADS) void k_start_words(Layout L, StartWord *words)
{
    __shared__ unsigned bits[TILE_WORDS];
    const int32_t tile = L.mixed_tiles[blockIdx.x];
    const int64_t tile_start = (int64_t)tile * TILE;
    const int32_t fb = L.tile_fb[tile], lb = L.tile_lb[tile];
    if (threadIdx.x < TILE_WORDS) bits[threadIdx.x] = threadIdx.x == 0 ? 1u : 0u;
    __syncthreads();
    for (int32_t b = fb + 1 + (int32_t)threadIdx.x; b <= lb; b += THREADS) {
        const int j = (int)(L.offs[b] - tile_start);
        atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    if (threadIdx.x < TILE_WORDS) {
        unsigned before = 0;
        for (unsigned i = 0; i < threadIdx.x; ++i) before += (unsigned)__popc(bits[i]);
        StartWord w;
        w.starts = bits[threadIdx.x];
        w.rank = before;
        words[(int64_t)blockIdx.x * TILE_WORDS + threadIdx.x] = w;
    }
}

}  // namespace ef
