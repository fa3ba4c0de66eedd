// Rules by which plan creation decides over a layout, apart from the tables themselves: plain C++, so that they can be
// checked without a GPU.
#pragma once
#include <stdint.h>

namespace ef {

constexpr int SMALL_SPAN = 256;         // most tiles of a block that spans tiles, in the kernels for small launches (ef_small.h)

// The same on a device that keeps `resident` workgroups of those kernels at once: a block's tiles wait for each other,
// so they have to be resident together, whatever part of the launch before them is still running.
inline int small_span(int resident)
{
    return resident / 2 < SMALL_SPAN ? resident / 2 : SMALL_SPAN;
}

// A mixed tile of few segments is taken like a whole one (compress_few), one of many by code of its own
// (compress_mixed, a "dense" tile).  The former's cost grows with the segments, for the server with a sum table for
// each, and beyond eight workers, where the others are added one by one, faster.  Layouts of such tiles
// alone, 20 M elements, server call, few / dense, us:
//   blocks of   2000 (4 segments)   820 (6)      600 (8)
//   2 workers   50.0 / 57.6         62 / 59      70 / 62
//   8 workers   50.6 / 74.8         63 / 76      71 / 79
//   16 workers  85.3 / 100          114 / 101    131 / 103
constexpr int FEW_SEGS = 16;            // most that compress_few takes
inline int few_segments(int max_workers) { return max_workers > 8 ? 5 : 6; }
// Where tiles of more segments are rare (a network's biases and norms between its smaller weights), one tile's
// cost is nothing beside what a dense one brings with it: the kernel that has the code for it, and p
// parked for a second pass where it meets a large block.  `between`: tiles of more than few_segments and at most
// FEW_SEGS.  Limit 6 / 16: bottleneck network of base 29 (1409 tiles, one of 7 to 9), server with 8
// workers 24.9 / 19.1 us, worker 28.5 / 26.1; transformer of width 230, server with 4 workers 26.1 / 22.2.
inline int few_segments(int max_workers, int64_t tiles, int64_t between)
{
    return between * 16 <= tiles ? FEW_SEGS : few_segments(max_workers);
}

// Where a tile of few segments comes in the order in which the kernels with one workgroup per tile take them: so many
// places ahead of its own, since it takes longer than a whole tile and its blocks wait for it.  Measured on the
// ResNet-50 layout (server, 7 workers) and on blocks of 64 tiles and 7 elements (worker, 7 workers): 0 60.4 / 590
// us, 128 57.1 / 590, 256 54.9 / 592, 512 53.6 / 596, 1024 56.9 / 607: far ahead, its slot is lost to the
// tiles it waits for.
constexpr int FEW_LEAD = 256;
// If a block that it ends has whole tiles before it (n tiles from t0 on, the first shared with another block or not),
// these wait for its part of the sum, and it goes ahead of them; but not of a block larger than `limit`, of which
// only the last tiles wait, if any (first_kept): a large block's end would stand thousands of places early, in a slot that
// waits for the block after it all the while.
inline int64_t few_place(int64_t tile, int64_t t0, int n, bool first_shared, int limit)
{
    const bool awaited = n - 1 - (first_shared ? 1 : 0) >= 1 && n <= limit;
    return (awaited ? t0 : tile) - FEW_LEAD;
}

// Does the server take two whole tiles of a block to a workgroup (k_server_tiles with PAIRS)?  many: more than eight workers.
// `mixed` of the layout's `tiles` are mixed ones, `between` lie in blocks that only pairs finish in one pass, and `resident`
// workgroups of the kernel with one tile to each run at once.  Server call, pairs / one tile, us:
//   up to eight workers, whole tiles and those of few segments: pairs, for any number of tiles (blocks of 64 tiles, 8 workers,
//   1200 tiles 12.4 / 12.2, 2400 16.3 / 19.4, 12 000 74.8 / 80.1); with dense ones where not all of it is resident
//   with one tile to a workgroup anyway (20 000 tiny blocks and four large ones, 1374 tiles 30.3 / 27.7, 2274 32.1 / 33.3)
//   more, with mixed tiles (9 workers; 16): 1788 26.0 / 25.3; 33.2 / 31.5, 2680 27.9 / 35.2; 34.4 / 46.4 (bottleneck networks),
//   19 469 156 / 189; 173 / 211 (a transformer, one tile of 400 mixed)
//   more, whole tiles alone or all but: one tile to a workgroup, but where most tiles are in blocks of 1025 to 1536 of them (six
//   of 1100, 54.4 / 75.0; 59.8 / 73.9).  That line is from before pairs had a table of the sums over twelve workers; today it would lie at the
//   tiles that are resident, too (blocks of 64: 1200 tiles 15.1 / 13.7; 15.6 / 11.9, 2400 19.1 / 21.2; 20.2 / 21.5, 12 000
//   77.7 / 87.4; 85.1 / 89.1, one ragged end, 5986 43.0 / 49.0; 47.3 / 51.7).
inline bool server_pairs(bool many, int64_t tiles, int64_t mixed, bool dense, int64_t between, int64_t resident)
{
    if (!many) return !dense || between > 0 || tiles > resident;
    return 3 * tiles > 4 * resident && (1024 * mixed >= tiles || 2 * between > tiles);
}

// A block larger than the one-pass limit has its first whole tiles parked (their p waits in memory for the scale) and keeps
// the last ones, about `keep` of them (0: none), in registers, as a one-pass block does.  How many of its `whole` tiles are
// parked: an even number, where any are kept (pairs are of one kind).
constexpr int parked_tiles(int whole, int keep)
{
    const int parked = whole > keep ? whole - keep : 0;
    return parked + (parked & 1) < whole ? parked + (parked & 1) : whole;
}
// The first tile that is kept; the whole ones start at `first_whole`.
constexpr int64_t first_kept(int64_t first_whole, int whole, int keep) { return first_whole + parked_tiles(whole, keep); }

// Parked tiles that are written out in step (sync_group_wait): `group` consecutive ones from the block's first whole tile
// on, fewer in the last group.  The last tile of a group is the one the others wait for, so it has to be a parked one, too:
// a kept tile never comes to that wait.
constexpr int64_t group_first(int64_t tile, int64_t first_whole, int group)
{
    return first_whole + (tile - first_whole) / group * group;
}
constexpr int64_t group_last(int64_t first, int group, int64_t first_kept)
{
    return first + group < first_kept ? first + group - 1 : first_kept - 1;
}

// What a workgroup whose wait ran out leaves for the one that ends the call (ef_tile.h, give_up): which segment, and of which call,
// so that nobody takes what another call left for its own.
constexpr unsigned long long PARKED_VALID = 1ull << 63;
constexpr unsigned long long PARKED_BOTH = 1ull << 62;      // the tile and the next one
constexpr unsigned long long PARKED_FORMS = 1ull << 61;     // the block's scale is still to be written, too
constexpr int PARKED_CALL_AT = 40, PARKED_SET_AT = 33;
constexpr unsigned PARKED_CALLS = 1u << 20, PARKED_SETS = 128u;
constexpr unsigned long long parked_entry(unsigned call, int set, int32_t tile, int slot, unsigned long long flags)
{
    return PARKED_VALID | flags | ((unsigned long long)(call % PARKED_CALLS) << PARKED_CALL_AT) | ((unsigned long long)set << PARKED_SET_AT) |
           ((unsigned long long)tile << 1) | (unsigned)slot;
}
constexpr bool parked_in(unsigned long long entry, unsigned call)
{
    return (entry & PARKED_VALID) && (unsigned)(entry >> PARKED_CALL_AT) % PARKED_CALLS == call % PARKED_CALLS;
}
constexpr int parked_set(unsigned long long entry) { return (int)((unsigned)(entry >> PARKED_SET_AT) % PARKED_SETS); }
constexpr int32_t parked_tile(unsigned long long entry) { return (int32_t)((entry >> 1) & 0xffffffffull); }
constexpr int parked_slot(unsigned long long entry) { return (int)(entry & 1ull); }
// Looks for the entry of `call` at most `polls` times.  load: what is there now; rest: between two looks.  0: it has not come.
template <class Load, class Rest>
constexpr unsigned long long await_parked(Load load, Rest rest, unsigned call, int polls)
{
    for (int n = 0; n < polls; ++n) {
        const unsigned long long entry = load();
        if (parked_in(entry, call)) return entry;
        rest();
    }
    return 0ull;
}

}  // namespace ef
