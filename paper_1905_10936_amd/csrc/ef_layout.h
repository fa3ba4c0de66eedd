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

}  // namespace ef
