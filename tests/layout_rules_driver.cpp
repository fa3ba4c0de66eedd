// Rules of csrc/ef_layout.h, checked on the host; built and run by tests/test_layout_rules.py.  Test infrastructure only.
#include "ef_layout.h"

#include <cstdio>
#include <initializer_list>

#define REQUIRE(cond)                                                  \
    do {                                                               \
        if (!(cond)) {                                                 \
            std::fprintf(stderr, "line %d: %s failed\n", __LINE__, #cond); \
            return 1;                                                  \
        }                                                              \
    } while (0)

int main()
{
    // a block's tiles fit twice over into what is resident, from a whole MI355X (256 units, two workgroups each) to
    // an eighth of one
    for (int units : {256, 128, 64, 32, 1}) {
        const int resident = 2 * units, span = ef::small_span(resident);
        REQUIRE(span >= 1 && 2 * span <= resident && span <= ef::SMALL_SPAN);
    }
    REQUIRE(ef::small_span(512) == ef::SMALL_SPAN);

    // no tile of more segments than compress_few has room for is taken as one of few; rare ones up to that are
    for (int workers : {1, 8, 9, 64})
        for (int64_t tiles : {1, 16, 1000})
            for (int64_t between : {0, 1, 60, 63, 1000}) {
                const int few = ef::few_segments(workers, tiles, between);
                REQUIRE(few <= ef::FEW_SEGS && few >= ef::few_segments(workers));
                REQUIRE((few == ef::FEW_SEGS) == (16 * between <= tiles));
            }
    REQUIRE(ef::few_segments(8) == 6 && ef::few_segments(9) == 5);
    // a tile where a block ends goes ahead of that block's whole tiles, but no further than what waits for it
    const int limit = 1024;
    for (int n : {1, 2, 3, 64, 1024, 1025, 12565, 300000})
        for (bool first_shared : {false, true}) {
            const int64_t tile = 1000000, t0 = tile - (n - 1), at = ef::few_place(tile, t0, n, first_shared, limit);
            const bool whole = n - 1 - (first_shared ? 1 : 0) >= 1;
            REQUIRE(at >= tile - ef::FEW_LEAD - limit);
            REQUIRE(at == (whole && n <= limit ? t0 : tile) - ef::FEW_LEAD);
        }
    std::puts("layout rules ok");
    return 0;
}
