// Host side of libef: plan construction, argument checks and kernel launches
// behind the C ABI declared in include/ef.h.
#include "ef.h"
#include "ef_debug.h"
#include "ef_device.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

struct ef_plan {
    ef::Layout L;
    ef::ScratchRef X;
    int max_workers;
    int device;
    int spin_limit;
    ef::CallState *d_state;         // [2]: calls made so far and the tags of the scratch sets, advanced on the device; a call's snapshot of it
    std::vector<int64_t> offs_host;
    std::vector<int32_t> fb_host, lb_host;
    // What depends on the one-pass limit, which differs between the kernels (each is bounded by what
    // the kernel's own grid keeps resident): role 0 = the persistent worker kernel, 1 = the server,
    // 2 = the worker kernel that runs one workgroup per tile.
    struct Role {
        int32_t fuse_limit, keep;   // see Layout
        bool beyond;                // there are blocks larger than fuse_limit
        uint32_t n_static;          // segments whose p the first kernels always park
        uint32_t n_late;            // blocks whose scale the first kernels never write
        uint32_t *d_static;         // [n_static]
        int32_t *d_late;            // [n_late]
        // deferred correction: position of every block in d_late if it is larger than fuse_limit, else -1 (written
        // while the mode is on); the whole tiles of those blocks (left out of d_static while the mode is on)
        int32_t *d_late_index;      // [B]
        int32_t *d_lazy_tiles;      // [n_lazy_tiles]
        uint32_t n_lazy_tiles;
    } role[3];
    int sync_group;                 // tiles of a large block that are written out in step (ef_plan_set_sync_group)
    int lazy;                       // deferred correction on (ef_plan_set_lazy)
    ef_state *state;                // the library-held state that lives on this plan, if any
    bool held;                      // a library-held state is, or is being, created
    // Host-side guard of the deferred mode: the residual buffers (workers, server) the last calls
    // left waiting for their correction, so that a call with other buffers is refused.  The
    // device-side CallState is what the kernels go by; this only catches misuse at the boundary.
    mutable const float *lazy_buf[2];
    mutable int64_t lazy_stride_seen;
    mutable bool phi_open;          // a diagnostics call has begun that did not come to its last kernel
    mutable int lazy_sets_seen;     // most workers any call since the last full flush has used
    float *d_lazy_scales;           // [nsets][lazy_stride]
    int lazy_stride;
    int32_t lim_persistent, lim_direct, lim_server;   // automatic limits
    int32_t user_fuse_limit;        // >= 0: set through ef_plan_tune, overrides the automatic limits
    // device memory owned by the plan: one allocation, and where its parts are
    void *d_arena;
    uint32_t *d_lists;              // the roles' d_static, d_late and d_lazy_tiles, one after the other
    int64_t *d_offs;
    int32_t *d_tile_fb;
    int32_t *d_tile_lb;
    unsigned long long *d_part;
    unsigned long long *d_ready;
    unsigned int *d_list_cnt;       // [CALL_WORDS]: defer_cnt[2], fin_cnt[2], ticket[2], lost_cnt[2] and the count of workgroups (alternating between calls)
    unsigned long long *d_parked;   // entries of segments parked in a call that ends without k_tail
    int worker_grid;                // workgroups of the persistent worker kernel
    int persistent;                 // worker: 1 pipelined persistent kernel, 0 one workgroup per tile
    int persistent_auto;            // what plan creation chose for this layout
    int persistent_forced;          // 1 after ef_plan_set_persistent(plan, 1): also for the momentum-free worker
    unsigned long long *d_defer_list;
    unsigned long long *d_fin_list;
    int32_t *d_mixed;               // tile lists
    int32_t *d_whole;
    ef::TileRec *d_tiles, *d_in_order, *d_paired, *d_mixed_recs;
    ef::StartWord *d_words;         // [n_mixed][TILE_WORDS]
    std::vector<char> dense_host;   // [ntiles] is the tile a dense one?
    std::vector<int32_t> mixed_host;
    // compressor-quality diagnostics
    int32_t *d_cross;               // blocks that span several tiles
    int32_t n_cross;
    double *d_qtile, *d_qpart;      // [max_workers][ntiles][2], [max_workers][2*ntiles][2]
    unsigned long long *d_phi;      // [max_workers] see QualityArgs
    unsigned *d_phi_done;
    // launches that (nearly) fit on the GPU all at once (ef_small.h)
    int small_wgs;                  // most workgroups such a launch may have
    int small_span;                 // most tiles of a block in it
    bool has_small;                 // this layout has such launches
    ef::SmallTile *d_small;         // [ntiles] records of the tiles, if it has
    ef::StartWord *d_small_words;   // [ntiles][TILE_WORDS]
    ef::SmallTables small;          // both
    bool kernels_auto;              // ef_plan_set_persistent has not been used to pick the kernels
    bool server_pairs[2];           // the server's calls (of up to eight workers, of more) take the whole tiles in pairs, if there are any
};

// Scratch of ef_compressor_quality_static: device memory that exists from the moment the library
// is loaded on a GPU, so that the call allocates nothing.  In host code the array's name is only a
// stand-in for the symbol; the memory is reached through the per-device address that
// static_scratch() looks up once per device.
static __device__ __align__(256) double scratch[(size_t)EF_QUALITY_STATIC_MAX_TILE_VECTORS * 6];

// Optimizer state held by the library (ef_state_create): Algorithm 4's m_i and e_i of n_workers
// workers and the server's e~, in device memory the caller never addresses, which lets every call
// on it run in the deferred-correction mode.
struct ef_state {
    ef_plan *plan;
    int n_workers;
    int64_t stride;                 // elements between two workers' rows: d rounded up to a multiple of 4
    float *mom, *err;               // [n_workers][stride]
    float *server_err;              // [d]
};

namespace {

enum { ROLE_TICKET = 0, ROLE_SERVER = 1, ROLE_TILES = 2 };

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[MAX_DEVICES];     // [device] address of `scratch` on that device, once looked up

thread_local char g_errbuf[512];
thread_local hipError_t g_last_hip = hipSuccess;

int hip_fail(hipError_t e)
{
    g_last_hip = e;
    return EF_ERR_HIP;
}

#define EF_HIP(call)                                  \
    do {                                              \
        hipError_t e_ = (call);                       \
        if (e_ != hipSuccess) return hip_fail(e_);    \
    } while (0)

// A plan's tables, scratch and state live on the device it was created on: a call made with another
// device current would launch kernels there on memory they cannot reach.
int on_plan_device(const ef_plan *plan)
{
    int device = -1;
    EF_HIP(hipGetDevice(&device));
    return device == plan->device ? EF_OK : EF_ERR_ARG;
}

// Address of the static scratch on the current device (which must be `device`).  The first call
// per device asks the runtime for the symbol's address; no memory is allocated.
int static_scratch(int device, double **out)
{
    if (device < 0 || device >= MAX_DEVICES) return EF_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol);
        g_scratch_ptr[device] = static_cast<double *>(ptr);
    }
    *out = g_scratch_ptr[device];
    return EF_OK;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Do the byte ranges [a, a + na) and [b, b + nb) share a byte?
bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + nb && b0 < a0 + na;
}

// Bytes spanned by n rows of `row` items that lie `stride` items apart (item size `item`).
size_t span_bytes(int n, int64_t stride, int64_t row, size_t item)
{
    return ((size_t)(n - 1) * (size_t)stride + (size_t)row) * item;
}

int check_offsets(const int64_t *offs, int64_t B)
{
    if (!offs) return EF_ERR_NULL;
    if (B < 1 || B > (int64_t)0x7fffffff - 1) return EF_ERR_OFFSETS;
    if (offs[0] != 0) return EF_ERR_OFFSETS;
    for (int64_t b = 0; b < B; ++b)
        if (offs[b + 1] <= offs[b]) return EF_ERR_OFFSETS;
    // tiles are indexed with 32-bit integers
    if ((offs[B] + ef::TILE - 1) / ef::TILE > (int64_t)0x7fffffff) return EF_ERR_OFFSETS;
    return EF_OK;
}

bool good_eta(float eta_prev, float eta)
{
    return std::isfinite(eta) && std::isfinite(eta_prev) && eta > 0.0f && eta_prev >= 0.0f;
}

void destroy_device(ef_plan *p)
{
    if (p->d_arena) (void)hipFree(p->d_arena);
}

// The parts of a plan's device memory: one allocation, one copy for the small tables and one for each
// large one, one fill (a plan used to make 30 allocations and 20 copies).
class Arena {
public:
    enum Fill { COPY, ZERO, LEAVE };
    template <class T>
    void add(T **where, size_t n, Fill fill, const T *from = nullptr)
    {
        parts_.push_back({reinterpret_cast<void **>(where), n * sizeof(T), fill, from});
    }
    // Allocates (the caller frees *base, also after an error) and sets every *where.
    int make(void **base)
    {
        const size_t align = 256, stage_max = 1u << 18;
        size_t total = 0, staged = 0, zero_from = 0, zero_to = 0;
        std::vector<Part *> order;
        for (int pass = 0; pass < 4; ++pass) {          // small tables, large tables, zeroed, the rest
            for (Part &q : parts_) {
                const int mine = q.fill == COPY ? (q.bytes <= stage_max ? 0 : 1) : q.fill == ZERO ? 2 : 3;
                if (mine != pass) continue;
                q.at = total;
                total += (q.bytes + align - 1) / align * align;
                order.push_back(&q);
            }
            if (pass == 0) staged = total;
            if (pass == 1) zero_from = total;
            if (pass == 2) zero_to = total;
        }
        std::vector<char> stage(staged, 0);
        EF_HIP(hipMalloc(base, total ? total : align));
        char *b = static_cast<char *>(*base);
        for (Part *q : order) {
            *q->where = b + q->at;
            if (q->fill != COPY || !q->bytes) continue;
            if (q->at < staged)
                memcpy(stage.data() + q->at, q->from, q->bytes);
            else
                EF_HIP(hipMemcpy(b + q->at, q->from, q->bytes, hipMemcpyHostToDevice));
        }
        if (staged) EF_HIP(hipMemcpy(b, stage.data(), staged, hipMemcpyHostToDevice));
        if (zero_to > zero_from) EF_HIP(hipMemset(b + zero_from, 0, zero_to - zero_from));
        return EF_OK;
    }

private:
    struct Part {
        void **where;
        size_t bytes;
        Fill fill;
        const void *from;
        size_t at = 0;
        Part(void **w, size_t n, Fill f, const void *p) : where(w), bytes(n), fill(f), from(p) {}
    };
    std::vector<Part> parts_;
};

// What plan creation asks the runtime about a device, once per device and process.
struct DeviceFacts {
    bool known;
    int cus;                                    // compute units
    int uniform, tiles, server[3], small;       // workgroups per unit of the kernels of these names (server: whole tiles, few, dense ones)
    int pairs[2];                               // of the server's with two tiles to a workgroup (up to eight workers, more)
    int server_many;                            // of the server's with one, for more than eight workers and tiles of few segments
};
DeviceFacts g_facts[MAX_DEVICES];

int device_facts(int device, DeviceFacts *out)
{
    if (device < 0 || device >= MAX_DEVICES) return EF_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    DeviceFacts &f = g_facts[device];
    if (!f.known) {
        int small_s = 0;
        EF_HIP(hipDeviceGetAttribute(&f.cus, hipDeviceAttributeMultiprocessorCount, device));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.uniform, ef::k_worker_uniform<true>, ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.tiles, (ef::k_worker_tiles<true, ef::ALL_WHOLE, false>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.server[0], (ef::k_server_tiles<ef::ALL_WHOLE, false, false>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.server[1], (ef::k_server_tiles<ef::FEW_TILES, false, false>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.server[2], (ef::k_server_tiles<ef::DENSE_TILES, false, false>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.server_many, (ef::k_server_tiles<ef::FEW_TILES, true, false>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.pairs[0], (ef::k_server_tiles<ef::DENSE_TILES, false, true>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.pairs[1], (ef::k_server_tiles<ef::DENSE_TILES, true, true>), ef::THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f.small, ef::k_worker_small<true>, ef::SMALL_THREADS, 0));
        EF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&small_s, ef::k_server_small, ef::SMALL_THREADS, 0));
        if (small_s < f.small) f.small = small_s;
        if (f.uniform < 1) f.uniform = 1;
        f.known = true;
    }
    *out = f;
    return EF_OK;
}

int64_t tiles_of_block(const ef_plan *p, int64_t b)
{
    const int64_t *o = p->offs_host.data();
    return (o[b + 1] - 1) / ef::TILE - o[b] / ef::TILE + 1;
}

bool has_uniform_tile(const ef_plan *p, int64_t b)
{
    const int64_t *o = p->offs_host.data();
    return tiles_of_block(p, b) - (o[b] % ef::TILE != 0 ? 1 : 0) - (o[b + 1] % ef::TILE != 0 ? 1 : 0) >= 1;
}

// A one-pass block without a whole tile is finished among the mixed tiles.  (Host mirror of
// finishes_with_mixed in ef_tile.h.)
bool finishes_with_mixed(const ef_plan *p, const ef_plan::Role &r, int64_t b)
{
    const int64_t n = tiles_of_block(p, b);
    return n >= 2 && n <= r.fuse_limit && !has_uniform_tile(p, b);
}

// What the main kernels of a call always leave to the kernel that ends it: the scales of the
// blocks larger than fuse_limit (in the deferred mode, or if they have no whole tile), and the residual of every open segment that is not finished
// where it is computed (the segments of those large blocks and, before the persistent worker kernel, the segments
// that blocks with whole tiles have in mixed tiles).  By blocks and mixed tiles, in ascending order: a loop over all tiles was
// a third of plan creation (16 384 whole tiles in blocks of 256: 260 -> 178 us with this and the pairs by runs).
int static_list(ef_plan *p, ef_plan::Role &r, std::vector<uint32_t> &all)
{
    std::vector<uint32_t> items;
    std::vector<int32_t> late, late_index, lazy_tiles;
    // are a block's segments in mixed tiles finished by the main kernels?
    const bool in_place = &r != &p->role[ROLE_TICKET];
    auto finished = [&](int64_t b, int32_t t) {
        return in_place && !p->dense_host[(size_t)t] ? tiles_of_block(p, b) <= r.fuse_limit : finishes_with_mixed(p, r, b);
    };
    const int64_t *o = p->offs_host.data();
    size_t m = 0;
    auto mixed_up_to = [&](int64_t end) {       // the segments in mixed tiles below `end` that have not come yet
        for (; m < p->mixed_host.size() && p->mixed_host[m] < end; ++m) {
            const int32_t t = p->mixed_host[m];
            const int64_t start = (int64_t)t * ef::TILE, fb = p->fb_host[t], lb = p->lb_host[t];
            if (o[fb] < start && !finished(fb, t)) items.push_back(((uint32_t)t << 1) | 0u);
            if (o[lb + 1] > start + ef::TILE && !finished(lb, t)) items.push_back(((uint32_t)t << 1) | 1u);
        }
    };
    if (p->lazy) late_index.assign((size_t)p->L.B, -1);
    r.keep = p->lazy ? 0 : r.fuse_limit;
    r.beyond = false;
    for (int64_t b = 0; b < p->L.B; ++b) {
        const int64_t n = tiles_of_block(p, b);
        if (n < 2 || n <= r.fuse_limit) continue;
        r.beyond = true;
        // a whole tile parks p only for these blocks, and their last whole tiles do not
        const int32_t first = (int32_t)(o[b] / ef::TILE) + (o[b] % ef::TILE != 0 ? 1 : 0);
        const int whole = (int)(o[b + 1] / ef::TILE) - first;
        const int32_t kept = whole < 1 ? first : (int32_t)ef::first_kept(first, whole, r.keep);
        mixed_up_to(first);
        for (int32_t t = first; t < kept; ++t) {
            if (p->lazy)
                lazy_tiles.push_back(t);        // deferred: corrected when the buffer is next loaded
            else
                items.push_back(((uint32_t)t << 1) | 0u);
        }
        if (r.keep > 0 && whole >= 1) continue;                 // its last whole tile forms the scale
        if (p->lazy && whole >= 1) late_index[(size_t)b] = (int32_t)late.size();
        late.push_back((int32_t)b);
    }
    mixed_up_to(p->L.ntiles);
    r.n_late = (uint32_t)late.size();
    r.n_static = (uint32_t)items.size();
    r.n_lazy_tiles = (uint32_t)lazy_tiles.size();
    if (p->lazy)
        EF_HIP(hipMemcpy(r.d_late_index, late_index.data(), sizeof(int32_t) * late_index.size(), hipMemcpyHostToDevice));
    r.d_static = p->d_lists + all.size();
    all.insert(all.end(), items.begin(), items.end());
    r.d_late = reinterpret_cast<int32_t *>(p->d_lists + all.size());
    all.insert(all.end(), late.begin(), late.end());
    r.d_lazy_tiles = reinterpret_cast<int32_t *>(p->d_lists + all.size());
    all.insert(all.end(), lazy_tiles.begin(), lazy_tiles.end());
    return EF_OK;
}

// Pick each role's one-pass limit and rebuild the lists that depend on it.
// Deferred mode, one workgroup per tile: blocks of up to this many tiles still wait for their
// scale in the kernel (measured: 6.6-6.75 ms on 2^28 elements and 8 workers for blocks of 2 to
// 64 tiles, as fast as anything else in that mode, and their residual is finished at once).
constexpr int32_t LAZY_WAIT_LIMIT = 64;

int refresh_limits_unguarded(ef_plan *p)
{
    auto clamp = [](int64_t v) { return (int32_t)(v < 0 ? 0 : (v > ef::FUSE_LIMIT_MAX ? ef::FUSE_LIMIT_MAX : v)); };
    ef_plan::Role &ticket = p->role[ROLE_TICKET], &server = p->role[ROLE_SERVER], &tiles = p->role[ROLE_TILES];
    if (p->user_fuse_limit >= 0) {
        ticket.fuse_limit = server.fuse_limit = tiles.fuse_limit = clamp(p->user_fuse_limit);
    } else if (p->lazy) {
        // With the correction deferred nothing has to wait for a block's scale.  The server and
        // the persistent worker kernel then run fastest without any wait; the worker kernel with
        // one workgroup per tile runs fastest when consecutive tiles are written out in step,
        // which small blocks get by waiting for their scale as usual and larger ones through
        // Layout::sync_group.  Both worker roles get the same limit: the buffers a call leaves
        // behind must fit the lists of whichever worker call comes next.
        ticket.fuse_limit = tiles.fuse_limit = p->persistent_forced ? 0 : LAZY_WAIT_LIMIT;
        // A layout of few tiles whose server residual the caller never sees is finished in one launch,
        // where waiting is cheap.
        server.fuse_limit = p->has_small && p->kernels_auto && p->held ? p->small_span : 0;
    } else {
        ticket.fuse_limit = clamp(p->lim_persistent);
        server.fuse_limit = clamp(p->lim_server);
        tiles.fuse_limit = clamp(p->lim_direct);
    }
    p->L.fuse_limit = p->role[0].fuse_limit;
    std::vector<uint32_t> all;
    for (auto &r : p->role) {
        int rc = static_list(p, r, all);
        if (rc) return rc;
    }
    if (!all.empty()) EF_HIP(hipMemcpy(p->d_lists, all.data(), sizeof(uint32_t) * all.size(), hipMemcpyHostToDevice));
    return EF_OK;
}

// The lists are built in host vectors: a failed allocation there becomes an error code, not an
// exception crossing the C boundary.
int refresh_limits(ef_plan *p)
{
    try {
        return refresh_limits_unguarded(p);
    } catch (const std::bad_alloc &) {
        return EF_ERR_ARG;
    }
}

// Records of the kernels for launches that (nearly) fit on the GPU all at once, if the
// layout has calls for them: few enough tiles, and no block of more tiles than a wavefront adds up, or than are
// sure to be resident together.
void small_tables(ef_plan *p, std::vector<ef::SmallTile> &out)
{
    const int32_t ntiles = p->L.ntiles;
    if (ntiles > p->small_wgs) return;
    const int64_t *o = p->offs_host.data();
    const int64_t d = p->L.d;
    for (int64_t b = 0; b < p->L.B; ++b)
        if (tiles_of_block(p, b) > p->small_span) return;
    out.resize((size_t)ntiles);
    p->has_small = true;
    for (int32_t t = 0; t < ntiles; ++t) {
        const int64_t start = (int64_t)t * ef::TILE, end = start + ef::TILE;
        const int32_t fb = p->fb_host[t], lb = p->lb_host[t];
        ef::SmallTile &r = out[(size_t)t];
        r = ef::SmallTile();
        r.fb = fb;
        r.nseg = lb - fb + 1;
        if (r.nseg > 1) p->small.words_of_tile = ef::TILE_WORDS;
        r.whole = fb == lb && end <= d;
        if (r.nseg <= ef::SMALL_BY_WAVE) {
            for (int i = 0; i < r.nseg; ++i) r.bound[i] = (int16_t)(o[fb + i] > start ? o[fb + i] - start : 0);
            r.bound[r.nseg] = (int16_t)((o[lb + 1] < end ? o[lb + 1] : end < d ? end : d) - start);
        }
        if (o[fb] < start || o[fb + 1] > end) {
            r.flags |= ef::SMALL_HEAD;
            r.head_t0 = (int32_t)(o[fb] / ef::TILE);
            r.head_n = (int32_t)tiles_of_block(p, fb);
            r.head_db = o[fb + 1] - o[fb];
            if (o[fb] % ef::TILE) r.flags |= ef::SMALL_HEAD_SLOT;
            if (o[fb + 1] <= end) r.flags |= ef::SMALL_WRITES_HEAD;
        }
        if (lb != fb && o[lb + 1] > end) {
            r.flags |= ef::SMALL_TAIL;
            r.tail_n = (int32_t)tiles_of_block(p, lb);
            r.tail_db = o[lb + 1] - o[lb];
        }
    }
}

int build_device(ef_plan *p)
{
    const int64_t B = p->L.B, d = p->L.d;
    const int32_t ntiles = p->L.ntiles;
    const int nsets = p->max_workers + 1;    // workers 0..max_workers-1, then the server
    std::vector<int32_t> &fb = p->fb_host, &lb = p->lb_host;
    fb.resize(ntiles);
    lb.resize(ntiles);
    {
        // block of the first and of the last valid element of every tile
        int64_t b = 0;
        const int64_t *o = p->offs_host.data();
        for (int32_t t = 0; t < ntiles; ++t) {
            const int64_t first = (int64_t)t * ef::TILE;
            int64_t last = first + ef::TILE - 1;
            if (last > d - 1) last = d - 1;
            while (o[b + 1] <= first) ++b;
            fb[t] = (int32_t)b;
            int64_t c = b;
            while (o[c + 1] <= last) ++c;
            lb[t] = (int32_t)c;
        }
    }
    EF_HIP(hipGetDevice(&p->device));
    DeviceFacts facts;
    { const int rc_facts = device_facts(p->device, &facts); if (rc_facts) return rc_facts; }
    // A block finishes in one pass if its tiles fit twice over into the tiles a kernel's workgroups hold at
    // once: grid x (PIPE_DEPTH + STAGE_DEPTH) for the persistent kernel, the resident workgroups for the
    // kernels that run one workgroup per tile (dispatched in grid order).  Larger limits were measured slower:
    // a block that fills most of the machine makes its first tiles wait for its last.  (The worker's is that of layouts of
    // whole tiles, 1024, for all: 57 % of what its kernel with dense tiles keeps resident.)
    p->worker_grid = facts.cus * facts.uniform;
    p->lim_persistent = (int32_t)((int64_t)p->worker_grid * (ef::PIPE_DEPTH + ef::STAGE_DEPTH) / 2);
    p->lim_direct = (int32_t)((int64_t)facts.cus * facts.tiles / 2);
    // Launches that (nearly) fit on the GPU all at once: up to twice what is resident.  A block's tiles are at
    // most half of what is resident and are dispatched in order, as the other one-pass kernels assume.  Measured, these
    // kernels / k_worker_tiles or k_server_tiles + k_tail, us, by tiles of one worker:
    //                                   64          512          1000
    //   worker, blocks of 30 000       9.2 / 13.0  11.2 / 15.1  21.5 / 20.8
    //   worker, blocks of 700          9.2 / 13.7  11.7 / 16.6  20.9 / 22.3
    //   server, 8 workers, of 30 000   8.9 / 12.0  12.3 / 13.3  20.8 / 16.1
    //   server, 8 workers, of 700      9.0 / 19.8  12.6 / 22.1  20.9 / 26.2
    //   server, 8 workers, 1 to 64 elements         13.6 / -    23.2 / 33.9
    // In the second round of workgroups the general kernels are ahead where all but a few tiles are whole, these
    // where they are not.
    p->small_wgs = 2 * facts.cus * facts.small;
    p->small_span = ef::small_span(facts.cus * facts.small);
    std::vector<ef::SmallTile> small;
    small_tables(p, small);

    std::vector<int32_t> &mixed = p->mixed_host;
    std::vector<int32_t> whole, cross;
    std::vector<ef::TileRec> tiles((size_t)ntiles);
    for (int32_t t = 0; t < ntiles; ++t) {
        const bool full = ((int64_t)t + 1) * ef::TILE <= d, one = fb[t] == lb[t] && full;
        const int64_t last_end = p->offs_host[(size_t)lb[t] + 1];
        const bool goes_on = lb[t] != fb[t] && last_end > ((int64_t)t + 1) * ef::TILE;
        const int32_t tail = goes_on ? (int32_t)(2 * tiles_of_block(p, lb[t]) + (last_end % ef::TILE != 0 ? 1 : 0)) : 0;
        const int64_t bs = p->offs_host[(size_t)fb[t]], be = p->offs_host[(size_t)fb[t] + 1];
        tiles[(size_t)t] = {t, fb[t], lb[t] - fb[t] + 1, one ? ef::TILE_ALONE : (int32_t)mixed.size(), tail, (int32_t)(bs / ef::TILE),
                            (int32_t)tiles_of_block(p, fb[t]), (int16_t)(bs % ef::TILE), (int16_t)(be % ef::TILE)};
        (one ? whole : mixed).push_back(t);
    }
    // Which mixed tiles are dense ones: those of many segments, and with one of them every tile that a block
    // without whole tiles shares with it, so that such a block is finished among tiles of one kind.
    std::vector<int32_t> dense;
    p->dense_host.assign((size_t)ntiles, 0);
    int64_t between = 0;
    for (int32_t t : mixed) {
        const int n = tiles[(size_t)t].nseg;
        between += n > ef::few_segments(p->max_workers) && n <= ef::FEW_SEGS;
    }
    const int few = ef::few_segments(p->max_workers, ntiles, between);
    for (int32_t t : mixed) p->dense_host[(size_t)t] = tiles[(size_t)t].nseg > few;
    auto joined = [&](int32_t t) {              // does a block without whole tiles go from tile t into t + 1?
        const int64_t b = lb[t];
        return t + 1 < ntiles && fb[t + 1] == b && tiles_of_block(p, b) == 2 && !has_uniform_tile(p, b);
    };
    for (int32_t t = 0; t + 1 < ntiles; ++t)
        if (p->dense_host[(size_t)t] && joined(t)) p->dense_host[(size_t)t + 1] = 1;
    for (int32_t t = ntiles - 1; t > 0; --t)
        if (p->dense_host[(size_t)t] && joined(t - 1)) p->dense_host[(size_t)t - 1] = 1;
    // Without whole tiles the layout runs one kernel, by the majority.
    if (whole.empty()) {
        int32_t n = 0;
        for (int32_t t : mixed) n += p->dense_host[(size_t)t];
        if (2 * n >= ntiles) p->dense_host.assign((size_t)ntiles, 1);
    }
    for (int32_t t : mixed)
        if (p->dense_host[(size_t)t]) {
            tiles[(size_t)t].nseg = -tiles[(size_t)t].nseg;
            dense.push_back(t);
        }
    p->L.n_dense = (int32_t)dense.size();
    p->L.n_grid = ntiles;
    // the server's limit is that of the kernel this layout runs, 1024 or, with dense tiles, 768 tiles on 256 units (8 workers; 2^28
    // elements in blocks of 1024 tiles: 560 us in one pass, 755 in two; twelve blocks of 850 tiles off the tile
    // boundaries: 87 and 119; with 100 000 tiny blocks among them 121 and 123, 16 workers 164 and 148)
    p->lim_server = (int32_t)((int64_t)facts.cus * facts.server[mixed.empty() ? 0 : dense.empty() ? 1 : 2] / 2);
    // The order in which the kernels with one workgroup per tile take the tiles: the dense ones, then the others
    // ascending, but for those of few segments (see few_place).  The limit for that is the one without pairs: the end of a
    // longer block keeps its place, also where pairs then take the block in one pass.
    const int awaited = p->lim_server > p->lim_direct ? p->lim_server : p->lim_direct;
    // And the same with the whole tiles of a block two by two, from its first on, for the server: where at least half of the
    // tiles are in pairs that wait for their block (one block of 2^28 elements, where few do: 462 us in pairs, 429 not), and
    // server_pairs says so.  Its limit is then half of the tiles that this kernel keeps resident, 1792 or 1536.  (Four
    // blocks of 2049 tiles among as many dense tiles, 4 workers: step 905 -> 893 us.)
    const bool many = p->max_workers > ef::SERVER_CHUNK;
    int32_t pair_limit = facts.cus * facts.pairs[many ? 1 : 0];
    int64_t pairs_only = 0;                     // tiles of blocks that one pass takes in pairs alone
    // the blocks that span several tiles
    for (int64_t b = 0; b < B; ++b) {
        const int64_t n = tiles_of_block(p, b);
        if (n < 2) continue;
        cross.push_back((int32_t)b);
        pairs_only += n > p->lim_server && n <= pair_limit ? n : 0;
    }
    p->server_pairs[0] = ef::server_pairs(false, ntiles, (int64_t)mixed.size(), !dense.empty(), pairs_only, (int64_t)facts.cus * facts.server[2]);
    p->server_pairs[1] = ef::server_pairs(true, ntiles, (int64_t)mixed.size(), !dense.empty(), pairs_only, (int64_t)facts.cus * facts.server_many);
    if (!p->server_pairs[many ? 1 : 0]) pair_limit = p->lim_server;     // fewer workers than the plan is for may still take pairs
    const bool may_pair = p->max_workers <= ef::PAIR_WORKERS && whole.size() * 2 >= (size_t)ntiles;
    std::vector<uint32_t> in_order, paired;
    double in_pairs = 0.0;                      // tiles in pairs that wait: of a block beyond the limit as large a part as would
    if (!mixed.empty()) in_order.reserve((size_t)ntiles);
    if (may_pair) paired.reserve((size_t)ntiles);
    size_t w = 0;
    auto whole_up_to = [&](int64_t end) {       // the whole tiles below `end` that have not come yet, block by block
        while (w < whole.size() && whole[w] < end) {
            const ef::TileRec &r = tiles[(size_t)whole[w]];
            // the block's whole tiles follow each other, from `first` to `last`
            const int32_t t = whole[w], first = r.t0 + (r.from != 0), last = r.t0 + r.n - 1 - (r.to != 0);
            const int32_t stop = last < end ? last + 1 : (int32_t)end;
            w += (size_t)(stop - t);
            if (!mixed.empty())
                for (int32_t i = t; i < stop; ++i) in_order.push_back((uint32_t)i);
            if (!may_pair) continue;
            int32_t i = t + ((t - first) & 1);
            int64_t pairs = 0;
            for (; i < stop && i < last; i += 2, ++pairs) paired.push_back((uint32_t)i | ef::PAIR_BIT);
            if (i < stop) paired.push_back((uint32_t)i);
            in_pairs += 2.0 * (double)pairs * (r.n <= pair_limit ? 1.0 : (double)pair_limit / (double)r.n);
        }
    };
    auto take = [&](int32_t t) {
        in_order.push_back((uint32_t)t);
        if (may_pair) paired.push_back((uint32_t)t);
    };
    for (int32_t t : dense) take(t);
    for (int32_t t : mixed) {
        const ef::TileRec &r = tiles[(size_t)t];
        if (r.nseg < 0) continue;
        whole_up_to(ef::few_place(t, r.t0, r.n, r.from != 0, awaited));
        take(t);
    }
    whole_up_to(ntiles);
    if (in_pairs * 2.0 < (double)ntiles)
        paired.clear();
    else
        p->lim_server = pair_limit;
    p->L.n_paired = (int32_t)paired.size();
    p->L.n_mixed = (int32_t)mixed.size();
    p->L.n_uniform = (int32_t)whole.size();
    // compressor-quality diagnostics: those blocks, and the per-tile sums
    p->n_cross = (int32_t)cross.size();

    const size_t nt = (size_t)ntiles, ns = (size_t)nsets, nv = (size_t)p->max_workers;
    // a block that crosses a tile boundary owns at least one of the 2*ntiles open segments
    const size_t max_cross = (size_t)(2 * (int64_t)ntiles < B ? 2 * (int64_t)ntiles : B);
    p->lazy_stride = (int)max_cross;
    Arena mem;
    mem.add(&p->d_offs, (size_t)B + 1, Arena::COPY, p->offs_host.data());
    mem.add(&p->d_tile_fb, nt, Arena::COPY, fb.data());
    mem.add(&p->d_tile_lb, nt, Arena::COPY, lb.data());
    mem.add(&p->d_mixed, mixed.size(), Arena::COPY, mixed.data());
    mem.add(&p->d_whole, whole.size(), Arena::COPY, whole.data());
    mem.add(&p->d_tiles, nt, Arena::COPY, tiles.data());
    // the records in grid order, in pairs and the mixed ones alone, one after the other
    const size_t n_in_order = in_order.size(), n_taken = n_in_order + paired.size() + mixed.size();
    in_order.insert(in_order.end(), paired.begin(), paired.end());
    in_order.insert(in_order.end(), mixed.begin(), mixed.end());
    // few of them travel with the small tables; many are taken on the device, where a launch costs less than the copy
    uint32_t *d_order = nullptr;
    std::vector<ef::TileRec> taken;
    if (n_taken <= 4096) {
        taken.reserve(n_taken);
        for (uint32_t i : in_order) {
            taken.push_back(tiles[i & ~ef::PAIR_BIT]);
            if (i & ef::PAIR_BIT) taken.back().words = ef::TILE_PAIR;
        }
        mem.add(&p->d_in_order, n_taken, Arena::COPY, taken.data());
    } else {
        mem.add(&d_order, n_taken, Arena::COPY, in_order.data());
        mem.add(&p->d_in_order, n_taken, Arena::LEAVE);
    }
    mem.add(&p->d_words, mixed.size() * ef::TILE_WORDS, Arena::LEAVE);
    mem.add(&p->d_cross, cross.size(), Arena::COPY, cross.data());
    mem.add(&p->d_part, 2 * nt * ns, Arena::ZERO);          // zeroed partial words carry tag 0
    // one 128-byte line per tile and set: a block's ready word sits in the line of its gatherer tile
    mem.add(&p->d_ready, (size_t)ef::READY_STRIDE * nt * ns, Arena::ZERO);
    mem.add(&p->d_list_cnt, ef::CALL_WORDS, Arena::ZERO);
    // an entry for a whole tile or pair, two for a mixed tile, in a call of at most ENDS_WGS_MAX workgroups
    const size_t max_parked = (whole.size() + 2 * mixed.size()) * nv, most_parked = 2 * (size_t)ef::ENDS_WGS_MAX;
    mem.add(&p->d_parked, max_parked < most_parked ? max_parked : most_parked, Arena::ZERO);
    mem.add(&p->d_state, 2, Arena::ZERO);
    mem.add(&p->d_lazy_scales, max_cross * ns, Arena::ZERO);
    mem.add(&p->d_defer_list, 2 * nt * ns, Arena::LEAVE);
    mem.add(&p->d_fin_list, max_cross * ns, Arena::LEAVE);
    mem.add(&p->d_lists, 3 * (3 * nt + max_cross), Arena::LEAVE);
    for (auto &r : p->role) mem.add(&r.d_late_index, (size_t)B, Arena::LEAVE);
    mem.add(&p->d_qpart, 4 * nt * nv, Arena::LEAVE);
    mem.add(&p->d_qtile, 2 * nt * nv, Arena::LEAVE);
    const std::vector<unsigned long long> ones(nv, 0x3ff0000000000000ull);      // 1.0
    mem.add(&p->d_phi, nv, Arena::COPY, ones.data());
    mem.add(&p->d_phi_done, nv, Arena::ZERO);
    if (p->has_small) {
        mem.add(&p->d_small, small.size(), Arena::COPY, small.data());
        mem.add(&p->d_small_words, p->small.words_of_tile ? nt * ef::TILE_WORDS : ef::TILE_WORDS, Arena::LEAVE);
    }
    { const int rc_mem = mem.make(&p->d_arena); if (rc_mem) return rc_mem; }
    p->L.mixed_tiles = p->d_mixed;
    p->L.whole_tiles = p->d_whole;
    p->L.tiles = p->d_tiles;
    p->L.grid_tiles = p->L.n_mixed ? p->d_in_order : p->d_tiles;
    p->d_paired = p->d_in_order + n_in_order;
    p->d_mixed_recs = p->d_paired + paired.size();
    p->L.paired_tiles = p->d_paired;
    if (d_order) {
        hipLaunchKernelGGL(ef::k_take_records, dim3((unsigned)((n_taken + ef::THREADS - 1) / ef::THREADS)), dim3(ef::THREADS), 0, nullptr,
                           (const ef::TileRec *)p->d_tiles, (const uint32_t *)d_order, (int)n_taken, p->d_in_order);
        EF_HIP(hipGetLastError());
    }
    p->L.words = p->d_words;
    p->L.mixed_recs = p->d_mixed_recs;
    p->L.offs = p->d_offs;
    p->L.tile_fb = p->d_tile_fb;
    p->L.tile_lb = p->d_tile_lb;
    p->X.part = p->d_part;
    p->X.ready = p->d_ready;
    p->X.defer_list = p->d_defer_list;
    p->X.fin_list = p->d_fin_list;
    p->X.list_cnt = p->d_list_cnt;
    p->X.state = p->d_state;
    p->X.snapshot = p->d_state + 1;
    p->X.step = p->d_state;
    p->X.parked = p->d_parked;
    p->X.lazy_scales = p->d_lazy_scales;
    p->X.lazy_stride = p->lazy_stride;
    if (p->has_small) {
        p->small.tiles = p->d_small;
        p->small.words = p->d_small_words;
    }
    if (p->small.words_of_tile) {
        hipLaunchKernelGGL(ef::k_small_words, dim3((unsigned)ntiles), dim3(ef::TILE_WORDS), 0, nullptr, p->L, p->d_small_words,
                           p->d_words);
        EF_HIP(hipGetLastError());
    } else if (p->L.n_mixed) {
        hipLaunchKernelGGL(ef::k_start_words, dim3((unsigned)p->L.n_mixed), dim3(ef::THREADS), 0, nullptr, p->L, p->d_words);
        EF_HIP(hipGetLastError());
    }
    p->user_fuse_limit = -1;
    // Which worker kernel for this layout.  The persistent kernel needs enough tiles per workgroup
    // to fill its pipeline; beyond that the choice follows the measured cost per tile of each
    // kernel by block size (2^28 elements, 8 workers, relative to the persistent kernel's 7.0 ms,
    // which does not depend on the block size up to its one-pass limit): the kernel with one
    // workgroup per tile is faster on blocks of up to 256 tiles, level up to 512, slower beyond,
    // and sends the first tiles of blocks above its own limit through the second pass.  (Such blocks are charged with two
    // passes over all of their tiles, as before their last ones were kept.)
    {
        const int64_t tiles_per_wg = (int64_t)p->L.n_uniform * p->max_workers / (p->worker_grid > 0 ? p->worker_grid : 1);
        const int64_t lim_hi = p->lim_persistent < ef::FUSE_LIMIT_MAX ? p->lim_persistent : ef::FUSE_LIMIT_MAX;
        const int64_t lim_lo = p->lim_direct < ef::FUSE_LIMIT_MAX ? p->lim_direct : ef::FUSE_LIMIT_MAX;
        double cost_direct = 0.0, cost_persistent = 0.0;
        for (int64_t b = 0; b < B; ++b) {
            const int64_t n = tiles_of_block(p, b);
            if (n < 2 || !has_uniform_tile(p, b)) continue;
            const double two_pass = 1.4;        // 28.125 instead of 20.125 bytes per element
            cost_persistent += (double)n * (n <= lim_hi ? 1.0 : two_pass);
            cost_direct += (double)n * (n > lim_lo ? two_pass - 0.03 : n <= 128 ? 0.94 : n <= 256 ? 0.98 : n <= 512 ? 1.0 : 1.05);
        }
        // a clear difference (blocks that only the persistent kernel finishes in one pass) decides from
        // 16 tiles per workgroup on, a small one only once the pipeline is well filled
        p->persistent_auto = ((tiles_per_wg >= 64 && cost_persistent < cost_direct) ||
                              (tiles_per_wg >= 16 && cost_persistent < 0.9 * cost_direct)) ? 1 : 0;
    }
    {
        double *unused = nullptr;       // the static scratch of this device, looked up once, ahead of the first call that needs it
        int rc_scratch = static_scratch(p->device, &unused);
        if (rc_scratch) return rc_scratch;
    }
    // Measured on an otherwise idle GPU: every wait of every benchmark layout ends within 64 polls
    // (about 0.3 us each); 2048 polls leave a factor of 32 for a GPU that is shared, and a wait that
    // is lost (its gatherer not resident) costs about 0.65 ms before the tile takes the second pass.
    p->spin_limit = 1 << 11;
    p->persistent = p->persistent_auto;
    p->persistent_forced = 0;
    int rc = refresh_limits(p);
    if (rc) return rc;
    EF_HIP(hipDeviceSynchronize());
    return EF_OK;
}

// Which worker kernel a call runs.  The persistent kernel (ROLE_TICKET) where plan creation or
// the caller chose it, with two exceptions.  The momentum-free worker moves 48 KiB per tile
// instead of 80: one ticket per tile would make the ticket counter (about 84 tickets per
// microsecond) its bottleneck, so it runs one workgroup per tile unless the persistent kernel
// was asked for explicitly.  And in the deferred mode the kernel with one workgroup per tile is
// the faster one (see refresh_limits).
int worker_role(const ef_plan *plan, bool has_mom)
{
    const bool ticketed = plan->L.n_uniform && plan->persistent &&
                          (plan->lazy ? plan->persistent_forced != 0 : (has_mom || plan->persistent_forced));
    return ticketed ? ROLE_TICKET : ROLE_TILES;
}

// Does a call over nsets sets go to the kernels of ef_small.h?  It has to be small enough, and no
// block may be left for a second pass (a limit set by the caller, or that of the deferred mode).
bool small_call(const ef_plan *plan, int role, int nsets)
{
    return plan->has_small && plan->kernels_auto && (int64_t)plan->L.ntiles * nsets <= plan->small_wgs &&
           !plan->role[role].beyond;
}

// Does the server's call over M workers take two whole tiles to a workgroup?
bool takes_pairs(const ef_plan *plan, int M)
{
    return plan->L.n_paired != 0 && plan->role[ROLE_SERVER].fuse_limit > 0 &&
           (!plan->kernels_auto || plan->server_pairs[M > ef::SERVER_CHUNK ? 1 : 0]);
}

// The updates, where nothing waits: as long as all of it is resident (with / without, weight decay, blocks of
// 32 768: 300 tiles 5.9 / 6.1 us, 700 8.6 / 8.4, 1000 11.6 / 11.2; blocks of 3000: 6.2 / 6.8, 9.1 / 8.9, 12.2 / 11.0).
bool small_update(const ef_plan *plan)
{
    return plan->has_small && plan->kernels_auto && 2 * (int64_t)plan->L.ntiles <= plan->small_wgs;
}

ef::ApplyTables apply_tables(const ef_plan *plan, bool small)
{
    return {plan->L.d, plan->L.W, plan->L.tiles, !small ? plan->L.words : plan->small.words_of_tile ? plan->small.words : nullptr};
}

// Scratch argument of one call over the sets [set_base, set_base + nsets).  Everything that
// differs between two calls of the same kind is read by the kernels from device memory.
struct CallScratch {
    ef::ScratchRef X;
};

CallScratch next_call(const ef_plan *plan, int set_base, int nsets)
{
    CallScratch c;
    c.X = plan->X;
    c.X.set_base = set_base;
    c.X.spin_limit = plan->spin_limit;
    c.X.ends = 0;
    c.X.nsets = nsets;
    c.X.lazy = plan->lazy;
    return c;
}

void ends_itself(CallScratch &c, int columns, float *err, int64_t err_stride, float *scales, int64_t scales_stride)
{
    c.X.ends = 1;
    c.X.columns = columns;
    c.X.err = err;
    c.X.err_stride = err_stride;
    c.X.scales = scales;
    c.X.scales_stride = scales_stride;
}

// Does the main kernel end the call, with `columns` workgroups to a set (ScratchRef::ends)?  Then nothing may be left for certain to
// a kernel after it, and what it has to hand on is set here.
bool main_kernel_ends(const ef_plan *plan, int role, CallScratch &c, int columns, float *err, int64_t err_stride, float *scales,
                      int64_t scales_stride)
{
    const ef_plan::Role &r = plan->role[role];
    if (role == ROLE_TICKET || r.n_static || r.n_late || (int64_t)columns * c.X.nsets > ef::ENDS_WGS_MAX) return false;
    ends_itself(c, columns, err, err_stride, scales, scales_stride);
    return true;
}

// The kernel after the main one(s): missing scales, parked residuals, and the step to the next call.
ef::Layout role_layout(const ef_plan *plan, int role)
{
    ef::Layout L = plan->L;
    L.fuse_limit = plan->role[role].fuse_limit;
    L.keep = plan->role[role].keep;
    L.lazy = plan->lazy;
    L.late_index = plan->role[role].d_late_index;
    L.sync_group = plan->sync_group;
    return L;
}

int launch_tail(const ef_plan *plan, int role, const CallScratch &c, int nsets, float *err, int64_t err_stride,
                float *scales, int64_t scales_stride, hipStream_t s)
{
    const ef_plan::Role &r = plan->role[role];
    const ef::Layout L = role_layout(plan, role);
    ef::TailArgs T;
    T.late_blocks = r.d_late;
    T.n_late = (int)r.n_late;
    T.items = r.d_static;
    T.n_items = (int)r.n_static;
    T.nsets = nsets;
    T.err = err;
    T.err_stride = err_stride;
    T.scales = scales;
    T.scales_stride = scales_stride;
    const int64_t n_fin = (int64_t)r.n_late * nsets, n_res = (int64_t)r.n_static * nsets;
    // a long list of parked segments is streamed by a kernel of its own, after this one has formed the scales
    const bool res_apart = n_res > ef::RES_IN_TAIL_MAX;
    if (res_apart) T.n_items = 0;
    T.fin_wgs = (int)(n_fin < ef::FIN_WGS_MAX ? n_fin : ef::FIN_WGS_MAX);
    T.res_wgs = res_apart ? 0 : (int)(n_res < ef::RES_WGS_MAX ? n_res : ef::RES_WGS_MAX);
    T.state = plan->d_state;
    T.lazy = plan->lazy;
    hipLaunchKernelGGL(ef::k_tail, dim3((unsigned)(T.fin_wgs + T.res_wgs + ef::DEFER_WGS)), dim3(ef::THREADS), 0, s, L,
                       c.X, T);
    EF_HIP(hipGetLastError());
    if (res_apart) {
        hipLaunchKernelGGL(ef::k_residual_static, dim3(r.n_static, (unsigned)nsets), dim3(ef::THREADS), 0, s, L,
                           (const uint32_t *)r.d_static, (int)r.n_static, err, err_stride, (const float *)scales,
                           scales_stride);
        EF_HIP(hipGetLastError());
    }
    return EF_OK;
}

// Bytes of one fused message: W sign words, then B fp32 scales, padded to 16.
size_t payload_bytes(const ef_plan *plan)
{
    const size_t raw = (size_t)plan->L.W * 8u + (size_t)plan->L.B * 4u;
    return (raw + 15u) / 16u * 16u;
}

int worker_step_impl(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *mom,
                     float *err, int64_t state_stride, float mu, float eta_prev, float eta, uint64_t *packed_signs,
                     int64_t signs_stride, float *scales, int64_t scales_stride, void *stream, double *quality = nullptr);
int server_step_impl(const ef_plan *plan, int M, const uint64_t *packed_signs, int64_t in_signs_stride,
                     const float *scales, int64_t in_scales_stride, float *server_err, float eta_prev, float eta,
                     uint64_t *out_signs, float *out_scales, void *stream);

}  // namespace

extern "C" {

size_t ef_sign_words(const ef_plan *plan) { return plan ? (size_t)plan->L.W : 0; }

int ef_plan_create(ef_plan **out, const int64_t *block_offsets_host, int64_t B, int max_workers, void *stream)
{
    (void)stream;
    if (!out) return EF_ERR_NULL;
    *out = nullptr;
    int rc = check_offsets(block_offsets_host, B);
    if (rc) return rc;
    if (max_workers < 1 || max_workers > EF_MAX_WORKERS) return EF_ERR_ARG;
    ef_plan *p = new (std::nothrow) ef_plan();
    if (!p) return EF_ERR_ARG;
    p->max_workers = max_workers;
    p->L.B = B;
    p->L.d = block_offsets_host[B];
    p->L.W = (p->L.d + 63) / 64;
    p->L.ntiles = (int32_t)((p->L.d + ef::TILE - 1) / ef::TILE);
    p->d_arena = nullptr;
    p->lazy = 0;
    p->state = nullptr;
    p->held = false;
    p->sync_group = 16;
    p->lazy_buf[0] = p->lazy_buf[1] = nullptr;
    p->lazy_stride_seen = 0;
    p->lazy_sets_seen = 0;
    for (auto &r : p->role) {
        r.n_static = r.n_late = r.n_lazy_tiles = 0;
        r.fuse_limit = r.keep = 0;
        r.beyond = false;
    }
    p->has_small = false;
    p->kernels_auto = true;

    try {
        p->offs_host.assign(block_offsets_host, block_offsets_host + B + 1);
        rc = build_device(p);
    } catch (const std::bad_alloc &) {      // host memory for the layout tables
        rc = EF_ERR_ARG;
    }
    if (rc) {
        destroy_device(p);
        delete p;
        return rc;
    }
    *out = p;
    return EF_OK;
}

int ef_plan_destroy(ef_plan *plan)
{
    if (!plan) return EF_ERR_NULL;
    if (plan->state) return EF_ERR_ARG;     // ef_state_destroy first
    (void)hipDeviceSynchronize();
    destroy_device(plan);
    delete plan;
    return EF_OK;
}

// Residual buffers whose large blocks still hold uncorrected p (deferred correction): the lists
// that say which blocks those are must not change under them.
static int residuals_pending(ef_plan *plan, bool *pending)
{
    ef::CallState st;
    EF_HIP(hipDeviceSynchronize());
    EF_HIP(hipMemcpy(&st, plan->d_state, sizeof st, hipMemcpyDeviceToHost));
    *pending = st.worker_pending != 0ull || st.server_pending != 0u;
    return EF_OK;
}

static int set_lazy(ef_plan *plan, int on);

int ef_plan_set_lazy(ef_plan *plan, int on)
{
    if (!plan) return EF_ERR_NULL;
    if (plan->state) return EF_ERR_ARG;     // a library-held state keeps the mode on
    return set_lazy(plan, on);
}

static int set_lazy(ef_plan *plan, int on)
{
    bool pending = false;
    int rc = residuals_pending(plan, &pending);
    if (rc) return rc;
    if (pending) return EF_ERR_ARG;
    plan->lazy = on ? 1 : 0;
    plan->lazy_buf[0] = plan->lazy_buf[1] = nullptr;
    plan->lazy_sets_seen = 0;
    return refresh_limits(plan);
}

int ef_plan_is_lazy(const ef_plan *plan) { return plan ? plan->lazy : 0; }

int ef_plan_set_sync_group(ef_plan *plan, int tiles)
{
    if (!plan) return EF_ERR_NULL;
    if (tiles < 0 || tiles > 256) return EF_ERR_ARG;
    EF_HIP(hipDeviceSynchronize());
    plan->sync_group = tiles;
    return EF_OK;
}

int ef_flush(const ef_plan *plan, int n_workers, float *err, int64_t state_stride, float *server_err, void *stream)
{
    if (!plan) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (err && (n_workers < 1 || n_workers > plan->max_workers ||
                (n_workers > 1 && (state_stride < plan->L.d || state_stride % 4))))
        return EF_ERR_ARG;
    if ((err && !aligned(err, 16)) || (server_err && !aligned(server_err, 16))) return EF_ERR_ALIGN;
    // other buffers than the ones that wait for their correction: refuse rather than corrupt them
    if (err && plan->lazy_buf[0] && (plan->lazy_buf[0] != err || plan->lazy_stride_seen != state_stride)) return EF_ERR_ARG;
    if (server_err && plan->lazy_buf[1] && plan->lazy_buf[1] != server_err) return EF_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int role = 0; role < 2; ++role) {
        float *buf = role == 0 ? err : server_err;
        if (!buf) continue;
        if (role == 1) {
            plan->lazy_buf[1] = nullptr;
        } else if (n_workers >= plan->lazy_sets_seen) {
            plan->lazy_buf[0] = nullptr;
            plan->lazy_sets_seen = 0;
        }
        const ef_plan::Role &r = plan->role[role == 0 ? ROLE_TILES : ROLE_SERVER];
        const int nsets = role == 0 ? n_workers : 1;
        const CallScratch c = next_call(plan, role == 0 ? 0 : plan->max_workers, nsets);
        if (r.n_lazy_tiles) {
            hipLaunchKernelGGL(ef::k_flush, dim3(r.n_lazy_tiles, (unsigned)nsets), dim3(ef::THREADS), 0, s,
                               role_layout(plan, role == 0 ? ROLE_TILES : ROLE_SERVER), c.X, (const int32_t *)r.d_lazy_tiles, (int)r.n_lazy_tiles, buf,
                               role == 0 ? state_stride : (int64_t)0);
            EF_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(ef::k_flush_done, dim3(1), dim3(64), 0, s, plan->d_state, c.X.set_base, nsets);
        EF_HIP(hipGetLastError());
    }
    return EF_OK;
}

int ef_plan_tune(ef_plan *plan, int fuse_limit, int spin_limit)
{
    if (!plan) return EF_ERR_NULL;
    if (spin_limit >= 0) plan->spin_limit = spin_limit;
    if (fuse_limit >= 0) {
        bool pending = false;
        int rc = residuals_pending(plan, &pending);
        if (rc) return rc;
        if (pending) return EF_ERR_ARG;
        plan->user_fuse_limit = fuse_limit;
        return refresh_limits(plan);
    }
    return EF_OK;
}

int ef_plan_fuse_limit(const ef_plan *plan)
{
    if (!plan) return 0;
    return plan->role[worker_role(plan, true)].fuse_limit;
}
int ef_plan_is_persistent(const ef_plan *plan)
{
    if (!plan) return 0;
    return plan->lazy ? (plan->persistent && plan->persistent_forced) : plan->persistent;
}

int ef_plan_last_fallbacks(ef_plan *plan, unsigned int *parked_tiles, unsigned int *late_blocks)
{
    if (!plan) return EF_ERR_NULL;
    EF_HIP(hipDeviceSynchronize());
    unsigned int cnt[8] = {};
    unsigned last = 0;
    ef::CallState st;
    EF_HIP(hipMemcpy(&st, plan->d_state, sizeof st, hipMemcpyDeviceToHost));
    if (st.calls > 0) {         // the most recent call used the counters of parity (calls - 1) & 1
        last = (st.calls - 1u) & 1u;
        EF_HIP(hipMemcpy(cnt, plan->d_list_cnt, sizeof cnt, hipMemcpyDeviceToHost));
    }
    if (parked_tiles) *parked_tiles = cnt[last] + cnt[6 + last];
    if (late_blocks) *late_blocks = cnt[2 + last];
    return EF_OK;
}

int ef_plan_set_persistent(ef_plan *plan, int on)
{
    if (!plan) return EF_ERR_NULL;
    bool pending = false;
    int rc = residuals_pending(plan, &pending);
    if (rc) return rc;
    if (pending) return EF_ERR_ARG;
    plan->persistent = on < 0 ? plan->persistent_auto : (on ? 1 : 0);
    plan->persistent_forced = on > 0 ? 1 : 0;
    plan->kernels_auto = on < 0;
    return refresh_limits(plan);
}

int ef_plan_small_calls(const ef_plan *plan, int n_workers)
{
    if (!plan || n_workers < 1) return 0;
    return (small_call(plan, ROLE_TILES, n_workers) ? 1 : 0) | (small_call(plan, ROLE_SERVER, 1) ? 2 : 0) |
           (small_update(plan) ? 4 : 0);
}

int ef_plan_server_pairs(const ef_plan *plan, int n_workers)
{
    return plan && n_workers >= 1 && n_workers <= plan->max_workers && !small_call(plan, ROLE_SERVER, 1) && takes_pairs(plan, n_workers);
}

int64_t ef_plan_d(const ef_plan *plan) { return plan ? plan->L.d : 0; }
int64_t ef_plan_blocks(const ef_plan *plan) { return plan ? plan->L.B : 0; }

int ef_worker_step(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *mom,
                   float *err, int64_t state_stride, float mu, float eta_prev, float eta,
                   uint64_t *packed_signs, float *scales, void *stream)
{
    if (!plan || !mom) return EF_ERR_NULL;
    return worker_step_impl(plan, n_workers, grad, grad_stride, mom, err, state_stride, mu, eta_prev, eta,
                            packed_signs, plan->L.W, scales, plan->L.B, stream);
}

int ef_worker_step_quality(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *mom,
                           float *err, int64_t state_stride, float mu, float eta_prev, float eta,
                           uint64_t *packed_signs, float *scales, double *quality, void *stream)
{
    if (!plan || !mom || !quality) return EF_ERR_NULL;
    return worker_step_impl(plan, n_workers, grad, grad_stride, mom, err, state_stride, mu, eta_prev, eta,
                            packed_signs, plan->L.W, scales, plan->L.B, stream, quality);
}

int ef_worker_step_sgd(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *err,
                       int64_t state_stride, float eta_prev, float eta, uint64_t *packed_signs, float *scales,
                       void *stream)
{
    if (!plan) return EF_ERR_NULL;
    return worker_step_impl(plan, n_workers, grad, grad_stride, nullptr, err, state_stride, 0.0f, eta_prev, eta,
                            packed_signs, plan->L.W, scales, plan->L.B, stream);
}

size_t ef_payload_bytes(const ef_plan *plan) { return plan ? payload_bytes(plan) : 0; }
size_t ef_payload_scales_offset(const ef_plan *plan) { return plan ? (size_t)plan->L.W * 8u : 0; }

int ef_worker_step_fused(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *mom,
                         float *err, int64_t state_stride, float mu, float eta_prev, float eta, void *payloads,
                         void *stream)
{
    if (!plan || !payloads || !mom) return EF_ERR_NULL;
    if (!aligned(payloads, 16)) return EF_ERR_ALIGN;
    const size_t pb = payload_bytes(plan);
    char *base = static_cast<char *>(payloads);
    return worker_step_impl(plan, n_workers, grad, grad_stride, mom, err, state_stride, mu, eta_prev, eta,
                            reinterpret_cast<uint64_t *>(base), (int64_t)(pb / 8u),
                            reinterpret_cast<float *>(base + (size_t)plan->L.W * 8u), (int64_t)(pb / 4u), stream);
}

int ef_server_step_fused(const ef_plan *plan, int M, const void *payloads, float *server_err, float eta_prev,
                         float eta, void *out_payload, void *stream)
{
    if (!plan || !payloads || !out_payload) return EF_ERR_NULL;
    if (!aligned(payloads, 16) || !aligned(out_payload, 16)) return EF_ERR_ALIGN;
    const size_t pb = payload_bytes(plan), so = (size_t)plan->L.W * 8u;
    if (M >= 1) {  // the output message may not overlap any input message
        const char *in0 = static_cast<const char *>(payloads), *o = static_cast<const char *>(out_payload);
        if (o < in0 + pb * (size_t)M && in0 < o + pb) return EF_ERR_ARG;
    }
    const char *in = static_cast<const char *>(payloads);
    char *out = static_cast<char *>(out_payload);
    return server_step_impl(plan, M, reinterpret_cast<const uint64_t *>(in), (int64_t)(pb / 8u),
                            reinterpret_cast<const float *>(in + so), (int64_t)(pb / 4u), server_err, eta_prev, eta,
                            reinterpret_cast<uint64_t *>(out), reinterpret_cast<float *>(out + so), stream);
}

int ef_apply_fused(const ef_plan *plan, float *params, const void *payload, float eta, void *stream)
{
    if (!plan || !payload) return EF_ERR_NULL;
    if (!aligned(payload, 16)) return EF_ERR_ALIGN;
    const char *in = static_cast<const char *>(payload);
    return ef_apply(plan, params, reinterpret_cast<const uint64_t *>(in),
                    reinterpret_cast<const float *>(in + (size_t)plan->L.W * 8u), eta, stream);
}

}  // extern "C"

namespace {

// The kernels of a diagnostics call between them keep a word of the plan for each vector (see QualityArgs::phi): from here to
// quality_end it is theirs.  After a call that has failed in between it has to be set again.
int quality_begin(const ef_plan *plan, hipStream_t s)
{
    if (plan->phi_open) {
        hipLaunchKernelGGL(ef::k_quality_reset, dim3(1), dim3(ef::THREADS), 0, s, plan->d_phi, plan->d_phi_done, plan->max_workers);
        EF_HIP(hipGetLastError());
    }
    plan->phi_open = true;
    return EF_OK;
}

int quality_end(const ef_plan *plan, const ef::QualityArgs &Q, int n_vectors, hipStream_t s)
{
    hipLaunchKernelGGL(ef::k_quality_blocks, dim3((unsigned)plan->n_cross + 1u, (unsigned)n_vectors), dim3(ef::THREADS), 0, s,
                       plan->L, Q, (const int32_t *)plan->d_cross, (int)plan->n_cross);
    EF_HIP(hipGetLastError());
    plan->phi_open = false;
    return EF_OK;
}

int worker_step_impl(const ef_plan *plan, int n_workers, const float *grad, int64_t grad_stride, float *mom,
                     float *err, int64_t state_stride, float mu, float eta_prev, float eta, uint64_t *packed_signs,
                     int64_t signs_stride, float *scales, int64_t scales_stride, void *stream, double *quality)
{
    // mom == nullptr selects Algorithm 3 (callers of the momentum entry points have checked theirs)
    const bool has_mom = mom != nullptr;
    if (!plan || !grad || !err || !packed_signs || !scales) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (n_workers < 1 || n_workers > plan->max_workers) return EF_ERR_ARG;
    if (!(mu >= 0.0f && mu < 1.0f) || !good_eta(eta_prev, eta)) return EF_ERR_ARG;
    // with one worker the strides are never used
    if (n_workers > 1 && (grad_stride < plan->L.d || state_stride < plan->L.d || grad_stride % 4 || state_stride % 4))
        return EF_ERR_ARG;
    {
        // in-place aliasing is the contract for mom and err only: nothing else may overlap
        const int64_t d = plan->L.d;
        const size_t g_bytes = span_bytes(n_workers, grad_stride, d, 4), s_bytes = span_bytes(n_workers, state_stride, d, 4);
        const size_t w_bytes = span_bytes(n_workers, signs_stride, plan->L.W, 8);
        const size_t c_bytes = span_bytes(n_workers, scales_stride, plan->L.B, 4);
        if (overlap(grad, g_bytes, err, s_bytes) || (has_mom && (overlap(grad, g_bytes, mom, s_bytes) ||
                                                                 overlap(mom, s_bytes, err, s_bytes))))
            return EF_ERR_ARG;
        const void *in[3] = {grad, err, mom};
        const size_t in_bytes[3] = {g_bytes, s_bytes, s_bytes};
        for (int k = 0; k < (has_mom ? 3 : 2); ++k)
            if (overlap(packed_signs, w_bytes, in[k], in_bytes[k]) || overlap(scales, c_bytes, in[k], in_bytes[k]))
                return EF_ERR_ARG;
    }
    if (!aligned(grad, 16) || (has_mom && !aligned(mom, 16)) || !aligned(err, 16) || !aligned(scales, 4) ||
        !aligned(packed_signs, 8))
        return EF_ERR_ALIGN;
    ef::WorkerArgs A;
    A.grad = grad;
    A.grad_stride = grad_stride;
    A.mom = mom;
    A.err = err;
    A.state_stride = state_stride;
    A.mu = mu;
    A.r = eta_prev / eta;
    A.signs = packed_signs;
    A.scales = scales;
    A.signs_stride = signs_stride;
    A.scales_stride = scales_stride;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (plan->lazy) {
        if (plan->lazy_buf[0] && (plan->lazy_buf[0] != err || plan->lazy_stride_seen != state_stride)) return EF_ERR_ARG;
        plan->lazy_buf[0] = err;
        plan->lazy_stride_seen = state_stride;
        if (n_workers > plan->lazy_sets_seen) plan->lazy_sets_seen = n_workers;
    }
    CallScratch c = next_call(plan, 0, n_workers);
    if (!quality && small_call(plan, ROLE_TILES, n_workers)) {
        const dim3 grid((unsigned)plan->L.ntiles, (unsigned)n_workers), block(ef::SMALL_THREADS);
        ends_itself(c, plan->L.ntiles, err, state_stride, scales, scales_stride);
        if (has_mom)
            hipLaunchKernelGGL(ef::k_worker_small<true>, grid, block, 0, s, plan->L, c.X, A, plan->small);
        else
            hipLaunchKernelGGL(ef::k_worker_small<false>, grid, block, 0, s, plan->L, c.X, A, plan->small);
        EF_HIP(hipGetLastError());
        return EF_OK;
    }
    const int role = quality ? (int)ROLE_TILES : worker_role(plan, has_mom);
    const ef::Layout L = role_layout(plan, role);
    // the kernels with dense and other tiles do not (server_ends)
    const bool ends = (!plan->L.n_dense || plan->L.n_dense == plan->L.ntiles) &&
                      main_kernel_ends(plan, role, c, plan->L.n_grid, err, state_stride, scales, scales_stride);
    if (quality) {
        if (!aligned(quality, 8)) return EF_ERR_ALIGN;
        const int rc_begin = quality_begin(plan, s);
        if (rc_begin) return rc_begin;
    }
    if (role == ROLE_TICKET) {
        // the mixed tiles first, in a kernel of their own, then the persistent kernel
        if (plan->L.n_mixed) {
            const dim3 grid((unsigned)plan->L.n_mixed, (unsigned)n_workers);
            if (has_mom)
                hipLaunchKernelGGL((ef::k_worker_mixed<true, false, false>), grid, dim3(ef::THREADS), 0, s, L, c.X, A, ef::QualityArgs());
            else
                hipLaunchKernelGGL((ef::k_worker_mixed<false, false, false>), grid, dim3(ef::THREADS), 0, s, L, c.X, A, ef::QualityArgs());
            EF_HIP(hipGetLastError());
        }
        int64_t wgs = (int64_t)plan->L.n_uniform * n_workers;
        if (wgs > plan->worker_grid) wgs = plan->worker_grid;
        const dim3 grid((unsigned)wgs), block(ef::THREADS);
        if (has_mom)
            hipLaunchKernelGGL(ef::k_worker_uniform<true>, grid, block, 0, s, L, c.X, A, n_workers);
        else
            hipLaunchKernelGGL(ef::k_worker_uniform<false>, grid, block, 0, s, L, c.X, A, n_workers);
        EF_HIP(hipGetLastError());
    } else {
        // every tile in one launch
        const dim3 grid((unsigned)plan->L.n_grid, (unsigned)n_workers), block(ef::THREADS);
        ef::QualityArgs Q;
        Q.v = nullptr;
        Q.stride = 0;
        Q.tile_sums = plan->d_qtile;
        Q.part_sums = plan->d_qpart;
        Q.out = quality;
        Q.phi = plan->d_phi;
        Q.done = plan->d_phi_done;
        const int kind = plan->L.n_dense ? 2 : plan->L.n_mixed ? 1 : 0;
        if (plan->L.n_dense == plan->L.ntiles) {
            typedef void (*Kernel)(ef::Layout, ef::ScratchRef, ef::WorkerArgs, ef::QualityArgs);
            static const Kernel kernels[3][2] = {{ef::k_worker_mixed<false, false, false>, ef::k_worker_mixed<false, false, true>},
                                                 {ef::k_worker_mixed<true, false, false>, ef::k_worker_mixed<true, false, true>},
                                                 {ef::k_worker_mixed<true, true, false>, ef::k_worker_mixed<true, true, true>}};
            hipLaunchKernelGGL(kernels[quality ? 2 : has_mom ? 1 : 0][ends], grid, block, 0, s, L, c.X, A, Q);
        } else if (quality && kind == 2)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::DENSE_TILES, true>), grid, block, 0, s, L, c.X, A, Q);
        else if (quality && kind == 1)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::FEW_TILES, true>), grid, block, 0, s, L, c.X, A, Q);
        else if (quality)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::ALL_WHOLE, true>), grid, block, 0, s, L, c.X, A, Q);
        else if (has_mom && kind == 2)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::DENSE_TILES, false>), grid, block, 0, s, L, c.X, A, Q);
        else if (has_mom && kind == 1)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::FEW_TILES, false>), grid, block, 0, s, L, c.X, A, Q);
        else if (has_mom)
            hipLaunchKernelGGL((ef::k_worker_tiles<true, ef::ALL_WHOLE, false>), grid, block, 0, s, L, c.X, A, Q);
        else if (kind == 2)
            hipLaunchKernelGGL((ef::k_worker_tiles<false, ef::DENSE_TILES, false>), grid, block, 0, s, L, c.X, A, Q);
        else if (kind == 1)
            hipLaunchKernelGGL((ef::k_worker_tiles<false, ef::FEW_TILES, false>), grid, block, 0, s, L, c.X, A, Q);
        else
            hipLaunchKernelGGL((ef::k_worker_tiles<false, ef::ALL_WHOLE, false>), grid, block, 0, s, L, c.X, A, Q);
        EF_HIP(hipGetLastError());
    }
    int rc = ends ? (int)EF_OK : launch_tail(plan, role, c, n_workers, err, state_stride, scales, scales_stride, s);
    if (rc || !quality) return rc;
    // the quality sums of the tiles are there: combine them per block and per vector
    ef::QualityArgs Q;
    Q.v = nullptr;
    Q.stride = 0;
    Q.tile_sums = plan->d_qtile;
    Q.part_sums = plan->d_qpart;
    Q.out = quality;
    Q.phi = plan->d_phi;
    Q.done = plan->d_phi_done;
    return quality_end(plan, Q, n_workers, s);
}

int server_step_impl(const ef_plan *plan, int M, const uint64_t *packed_signs, int64_t in_signs_stride,
                     const float *scales, int64_t in_scales_stride, float *server_err, float eta_prev, float eta,
                     uint64_t *out_signs, float *out_scales, void *stream)
{
    if (!plan || !packed_signs || !scales || !server_err || !out_signs || !out_scales) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (M < 1 || M > plan->max_workers) return EF_ERR_ARG;
    if (!good_eta(eta_prev, eta)) return EF_ERR_ARG;
    {
        // the server residual is updated in place; the payloads may overlap neither it nor each other
        const size_t in_w = span_bytes(M, in_signs_stride, plan->L.W, 8), in_c = span_bytes(M, in_scales_stride, plan->L.B, 4);
        const size_t out_w = (size_t)plan->L.W * 8u, out_c = (size_t)plan->L.B * 4u, e_bytes = (size_t)plan->L.d * 4u;
        if (overlap(out_signs, out_w, packed_signs, in_w) || overlap(out_signs, out_w, scales, in_c) ||
            overlap(out_scales, out_c, packed_signs, in_w) || overlap(out_scales, out_c, scales, in_c) ||
            overlap(out_signs, out_w, out_scales, out_c))
            return EF_ERR_ARG;
        if (overlap(server_err, e_bytes, packed_signs, in_w) || overlap(server_err, e_bytes, scales, in_c) ||
            overlap(server_err, e_bytes, out_signs, out_w) || overlap(server_err, e_bytes, out_scales, out_c))
            return EF_ERR_ARG;
    }
    if (!aligned(server_err, 16) || !aligned(packed_signs, 8) || !aligned(out_signs, 8) ||
        !aligned(scales, 4) || !aligned(out_scales, 4))
        return EF_ERR_ALIGN;
    ef::ServerArgs A;
    A.M = M;
    A.signs_in = packed_signs;
    A.scales_in = scales;
    A.in_signs_stride = in_signs_stride;
    A.in_scales_stride = in_scales_stride;
    A.err = server_err;
    A.r = eta_prev / eta;
    A.Mf = (float)M;
    A.Minv = (M & (M - 1)) == 0 ? 1.0f / (float)M : 0.0f;
    A.signs = out_signs;
    A.scales = out_scales;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (plan->lazy) {
        if (plan->lazy_buf[1] && plan->lazy_buf[1] != server_err) return EF_ERR_ARG;
        plan->lazy_buf[1] = server_err;
    }
    CallScratch c = next_call(plan, plan->max_workers, 1);
    if (small_call(plan, ROLE_SERVER, 1)) {
        ends_itself(c, plan->L.ntiles, server_err, 0, out_scales, 0);
        hipLaunchKernelGGL(ef::k_server_small, dim3((unsigned)plan->L.ntiles), dim3(ef::SMALL_THREADS), 0, s, plan->L, c.X, A,
                           plan->small, plan->max_workers);
        EF_HIP(hipGetLastError());
        return EF_OK;
    }
    const ef::Layout L = role_layout(plan, ROLE_SERVER);
    const dim3 block(ef::THREADS);
    const int kind = L.n_dense ? 2 : L.n_mixed ? 1 : 0;
    const bool many = M > ef::SERVER_CHUNK, pairs = takes_pairs(plan, M);
    const bool ends = (L.n_dense == L.ntiles || ef::server_ends(kind, many, pairs)) && main_kernel_ends(plan, ROLE_SERVER, c, pairs ? L.n_paired : L.n_grid, server_err, 0, out_scales, 0);
    if (L.n_dense == L.ntiles) {
        hipLaunchKernelGGL(ef::k_server_mixed, dim3((unsigned)L.n_grid), block, 0, s, L, c.X, A, plan->max_workers);
    } else {
        typedef void (*Kernel)(ef::Layout, ef::ScratchRef, ef::ServerArgs, int);
        static const Kernel kernels[2][2][3] = {
            {{ef::k_server_tiles<0, false, false>, ef::k_server_tiles<1, false, false>, ef::k_server_tiles<2, false, false>},
             {ef::k_server_tiles<0, true, false>, ef::k_server_tiles<1, true, false>, ef::k_server_tiles<2, true, false>}},
            {{ef::k_server_tiles<0, false, true>, ef::k_server_tiles<1, false, true>, ef::k_server_tiles<2, false, true>},
             {ef::k_server_tiles<0, true, true>, ef::k_server_tiles<1, true, true>, ef::k_server_tiles<2, true, true>}}};
        hipLaunchKernelGGL(kernels[pairs][many][kind], dim3((unsigned)(pairs ? L.n_paired : L.n_grid)), block, 0, s, L, c.X, A,
                           plan->max_workers);
    }
    EF_HIP(hipGetLastError());
    if (ends) return EF_OK;
    return launch_tail(plan, ROLE_SERVER, c, 1, server_err, (int64_t)0, out_scales, (int64_t)0, s);
}

}  // namespace

extern "C" {

int ef_server_step(const ef_plan *plan, int M, const uint64_t *packed_signs, const float *scales,
                   float *server_err, float eta_prev, float eta, uint64_t *out_signs, float *out_scales,
                   void *stream)
{
    if (!plan) return EF_ERR_NULL;
    return server_step_impl(plan, M, packed_signs, plan->L.W, scales, plan->L.B, server_err, eta_prev, eta,
                            out_signs, out_scales, stream);
}

int ef_apply(const ef_plan *plan, float *params, const uint64_t *packed_signs, const float *scales, float eta,
             void *stream)
{
    if (!plan || !params || !packed_signs || !scales) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (!(std::isfinite(eta) && eta > 0.0f)) return EF_ERR_ARG;
    if (!aligned(params, 16) || !aligned(packed_signs, 8) || !aligned(scales, 4)) return EF_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    dim3 grid((unsigned)plan->L.ntiles, 1u);
    if (small_update(plan))
        hipLaunchKernelGGL(ef::k_apply_small<false>, grid, dim3(ef::SMALL_THREADS), 0, s, apply_tables(plan, true), params,
                           (float *)nullptr, packed_signs, scales, eta, 0.0f, 0.0f);
    else
        hipLaunchKernelGGL(ef::k_apply, grid, dim3(ef::THREADS), 0, s, apply_tables(plan, false), params, packed_signs, scales, eta);
    EF_HIP(hipGetLastError());
    return EF_OK;
}

int ef_apply_wd(const ef_plan *plan, float *params, float *decay_mom, const uint64_t *packed_signs,
                const float *scales, float eta, float mu, float lambda, void *stream)
{
    if (!plan || !params || !decay_mom || !packed_signs || !scales) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (!(std::isfinite(eta) && eta > 0.0f)) return EF_ERR_ARG;
    if (!(mu >= 0.0f && mu < 1.0f)) return EF_ERR_ARG;
    if (!(std::isfinite(lambda) && lambda >= 0.0f)) return EF_ERR_ARG;
    if (!aligned(params, 16) || !aligned(decay_mom, 16) || !aligned(packed_signs, 8) || !aligned(scales, 4))
        return EF_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    dim3 grid((unsigned)plan->L.ntiles, 1u);
    if (small_update(plan))
        hipLaunchKernelGGL(ef::k_apply_small<true>, grid, dim3(ef::SMALL_THREADS), 0, s, apply_tables(plan, true), params,
                           decay_mom, packed_signs, scales, eta, mu, lambda);
    else
        hipLaunchKernelGGL(ef::k_apply_wd, grid, dim3(ef::THREADS), 0, s, apply_tables(plan, false), params, decay_mom, packed_signs,
                           scales, eta, mu, lambda);
    EF_HIP(hipGetLastError());
    return EF_OK;
}

static int quality_launch(const ef_plan *plan, int n_vectors, const float *v, int64_t stride, double *out,
                          double *tile_sums, double *part_sums, hipStream_t s)
{
    ef::QualityArgs Q;
    Q.v = v;
    Q.stride = stride;
    Q.tile_sums = tile_sums;
    Q.part_sums = part_sums;
    Q.out = out;
    Q.phi = plan->d_phi;
    Q.done = plan->d_phi_done;
    const int rc = quality_begin(plan, s);
    if (rc) return rc;
    hipLaunchKernelGGL(ef::k_quality_tiles, dim3((unsigned)plan->L.ntiles, (unsigned)n_vectors), dim3(ef::THREADS), 0,
                       s, plan->L, Q);
    EF_HIP(hipGetLastError());
    return quality_end(plan, Q, n_vectors, s);
}

static int quality_args(const ef_plan *plan, int n_vectors, const float *v, int64_t stride, const double *out)
{
    if (!plan || !v || !out) return EF_ERR_NULL;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if (n_vectors < 1 || n_vectors > plan->max_workers) return EF_ERR_ARG;
    if (n_vectors > 1 && (stride < plan->L.d || stride % 4)) return EF_ERR_ARG;
    if (!aligned(v, 16) || !aligned(out, 8)) return EF_ERR_ALIGN;
    return EF_OK;
}

int ef_compressor_quality(ef_plan *plan, int n_vectors, const float *v, int64_t stride, double *out, void *stream)
{
    const int rc = quality_args(plan, n_vectors, v, stride, out);
    if (rc) return rc;
    return quality_launch(plan, n_vectors, v, stride, out, plan->d_qtile, plan->d_qpart, static_cast<hipStream_t>(stream));
}

int ef_compressor_quality_static(const ef_plan *plan, int n_vectors, const float *v, int64_t stride, double *out,
                                 void *stream)
{
    int rc = quality_args(plan, n_vectors, v, stride, out);
    if (rc) return rc;
    const int64_t tile_vectors = (int64_t)plan->L.ntiles * n_vectors;
    if (tile_vectors > (int64_t)EF_QUALITY_STATIC_MAX_TILE_VECTORS) return EF_ERR_SIZE;
    double *base = nullptr;
    rc = static_scratch(plan->device, &base);      // quality_args has checked that the plan's device is current
    if (rc) return rc;
    // [n][ntiles][2] tile sums, then [n][2*ntiles][2] sums of open segments; every word the kernels read
    // is written earlier in the same call, so nothing has to be cleared
    return quality_launch(plan, n_vectors, v, stride, out, base, base + 2 * tile_vectors, static_cast<hipStream_t>(stream));
}

int ef_state_create(ef_plan *plan, int n_workers, ef_state **out, void *stream)
{
    if (!plan || !out) return EF_ERR_NULL;
    *out = nullptr;
    if (n_workers < 1 || n_workers > plan->max_workers || plan->state) return EF_ERR_ARG;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    plan->held = true;
    int rc = set_lazy(plan, 1);             // refused (EF_ERR_ARG) while caller-owned buffers wait for a correction
    ef_state *st = rc ? nullptr : new (std::nothrow) ef_state();
    if (!st) {
        plan->held = false;
        if (rc) return rc;
        (void)set_lazy(plan, 0);
        return EF_ERR_ARG;
    }
    st->plan = plan;
    st->n_workers = n_workers;
    st->stride = (plan->L.d + 3) / 4 * 4;
    st->mom = st->err = st->server_err = nullptr;
    const size_t rows = sizeof(float) * (size_t)st->stride * (size_t)n_workers, one = sizeof(float) * (size_t)plan->L.d;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipMalloc(&st->mom, rows);
    if (e == hipSuccess) e = hipMalloc(&st->err, rows);
    if (e == hipSuccess) e = hipMalloc(&st->server_err, one);
    // m_0 = e_0 = e~_0 = 0 (Algorithm 4, input line)
    if (e == hipSuccess) e = hipMemsetAsync(st->mom, 0, rows, s);
    if (e == hipSuccess) e = hipMemsetAsync(st->err, 0, rows, s);
    if (e == hipSuccess) e = hipMemsetAsync(st->server_err, 0, one, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        if (st->mom) (void)hipFree(st->mom);
        if (st->err) (void)hipFree(st->err);
        if (st->server_err) (void)hipFree(st->server_err);
        delete st;
        plan->held = false;
        (void)set_lazy(plan, 0);
        return hip_fail(e);
    }
    plan->state = st;
    *out = st;
    return EF_OK;
}

int ef_state_destroy(ef_state *state)
{
    if (!state) return EF_ERR_NULL;
    ef_plan *plan = state->plan;
    (void)hipDeviceSynchronize();
    (void)hipFree(state->mom);
    (void)hipFree(state->err);
    (void)hipFree(state->server_err);
    plan->state = nullptr;
    delete state;
    // the buffers that waited for a correction are gone: clear the marks, leave the mode
    hipLaunchKernelGGL(ef::k_flush_done, dim3(1), dim3(64), 0, nullptr, plan->d_state, 0, plan->max_workers);
    hipLaunchKernelGGL(ef::k_flush_done, dim3(1), dim3(64), 0, nullptr, plan->d_state, plan->max_workers, 1);
    EF_HIP(hipGetLastError());
    plan->lazy_buf[0] = plan->lazy_buf[1] = nullptr;
    plan->lazy_sets_seen = 0;
    plan->held = false;
    return set_lazy(plan, 0);
}

int ef_worker_step_state(const ef_plan *plan, ef_state *state, const float *grad, int64_t grad_stride, float mu,
                         float eta_prev, float eta, uint64_t *packed_signs, float *scales, void *stream)
{
    if (!plan || !state) return EF_ERR_NULL;
    if (state->plan != plan) return EF_ERR_ARG;
    return worker_step_impl(plan, state->n_workers, grad, grad_stride, state->mom, state->err, state->stride, mu,
                            eta_prev, eta, packed_signs, plan->L.W, scales, plan->L.B, stream);
}

int ef_server_step_state(const ef_plan *plan, ef_state *state, int M, const uint64_t *packed_signs, const float *scales,
                         float eta_prev, float eta, uint64_t *out_signs, float *out_scales, void *stream)
{
    if (!plan || !state) return EF_ERR_NULL;
    if (state->plan != plan) return EF_ERR_ARG;
    return server_step_impl(plan, M, packed_signs, plan->L.W, scales, plan->L.B, state->server_err, eta_prev, eta,
                            out_signs, out_scales, stream);
}

// Copies between the library-held state and caller buffers, row by row (the strides may differ).
static int copy_state(const ef_plan *plan, ef_state *state, float *mom, float *err, int64_t state_stride,
                      float *server_err, bool to_caller, hipStream_t s)
{
    const size_t row = sizeof(float) * (size_t)plan->L.d;
    const size_t mine = sizeof(float) * (size_t)state->stride, theirs = sizeof(float) * (size_t)state_stride;
    float *pairs[2][2] = {{state->mom, mom}, {state->err, err}};
    for (auto &pr : pairs) {
        if (!pr[1]) continue;
        if (to_caller)
            EF_HIP(hipMemcpy2DAsync(pr[1], theirs, pr[0], mine, row, (size_t)state->n_workers, hipMemcpyDeviceToDevice, s));
        else
            EF_HIP(hipMemcpy2DAsync(pr[0], mine, pr[1], theirs, row, (size_t)state->n_workers, hipMemcpyDeviceToDevice, s));
    }
    if (server_err) {
        if (to_caller)
            EF_HIP(hipMemcpyAsync(server_err, state->server_err, row, hipMemcpyDeviceToDevice, s));
        else
            EF_HIP(hipMemcpyAsync(state->server_err, server_err, row, hipMemcpyDeviceToDevice, s));
    }
    return EF_OK;
}

static int state_copy_args(const ef_plan *plan, const ef_state *state, const float *mom, const float *err,
                           int64_t state_stride, const float *server_err)
{
    if (!plan || !state) return EF_ERR_NULL;
    if (state->plan != plan) return EF_ERR_ARG;
    { const int rc_dev = on_plan_device(plan); if (rc_dev) return rc_dev; }
    if ((mom || err) && state->n_workers > 1 && state_stride < plan->L.d) return EF_ERR_ARG;
    if ((mom && !aligned(mom, 4)) || (err && !aligned(err, 4)) || (server_err && !aligned(server_err, 4))) return EF_ERR_ALIGN;
    return EF_OK;
}

int ef_state_export(const ef_plan *plan, ef_state *state, float *mom, float *err, int64_t state_stride,
                    float *server_err, void *stream)
{
    int rc = state_copy_args(plan, state, mom, err, state_stride, server_err);
    if (rc) return rc;
    // write the corrections that are still waiting, then the buffers hold m, e and e~ of Algorithm 4
    rc = ef_flush(plan, state->n_workers, state->err, state->stride, state->server_err, stream);
    if (rc) return rc;
    return copy_state(plan, state, mom, err, state_stride, server_err, true, static_cast<hipStream_t>(stream));
}

int ef_state_import(const ef_plan *plan, ef_state *state, const float *mom, const float *err, int64_t state_stride,
                    const float *server_err, void *stream)
{
    int rc = state_copy_args(plan, state, mom, err, state_stride, server_err);
    if (rc) return rc;
    // what is brought in is finished state: no correction may be left waiting for the buffers it replaces
    rc = ef_flush(plan, state->n_workers, err ? state->err : nullptr, state->stride, server_err ? state->server_err : nullptr,
                  stream);
    if (rc) return rc;
    return copy_state(plan, state, const_cast<float *>(mom), const_cast<float *>(err), state_stride,
                      const_cast<float *>(server_err), false, static_cast<hipStream_t>(stream));
}

const char *ef_strerror(int code)
{
    const char *t;
    switch (code) {
    case EF_OK: t = "ok"; break;
    case EF_ERR_NULL: t = "a required pointer is NULL"; break;
    case EF_ERR_OFFSETS: t = "block_offsets is not a partition (0 = o[0] < o[1] < ... < o[B] = d)"; break;
    case EF_ERR_ARG: t = "argument out of range"; break;
    case EF_ERR_ALIGN: t = "pointer not aligned (fp32 arrays 16 bytes, sign words 8 bytes)"; break;
    case EF_ERR_SIZE:
        t = "input too large for the static scratch of ef_compressor_quality_static (tiles x vectors above "
            "EF_QUALITY_STATIC_MAX_TILE_VECTORS): use ef_compressor_quality";
        break;
    case EF_ERR_HIP:
        snprintf(g_errbuf, sizeof g_errbuf, "HIP runtime error: %s", hipGetErrorString(g_last_hip));
        return g_errbuf;
    default: t = "unknown error code"; break;
    }
    snprintf(g_errbuf, sizeof g_errbuf, "%s", t);
    return g_errbuf;
}

}  // extern "C"
