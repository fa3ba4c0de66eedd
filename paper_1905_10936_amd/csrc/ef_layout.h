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

}  // namespace ef
