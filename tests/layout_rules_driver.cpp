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
    // server, two tiles to a workgroup or one: the layouts on both sides of each line of the rule
    const int64_t dense_resident = 1536, many_resident = 1792;
    for (int64_t tiles : {300, 1536, 1537, 90000}) {
        REQUIRE(ef::server_pairs(false, tiles, 0, false, 0, dense_resident));
        REQUIRE(ef::server_pairs(false, tiles, 60, true, 0, dense_resident) == (tiles > dense_resident));
        REQUIRE(ef::server_pairs(false, tiles, 60, true, 1100, dense_resident));
    }
    for (int64_t tiles : {300, 2389, 2390, 30000}) {
        const bool large = tiles > many_resident * 4 / 3;
        REQUIRE(!ef::server_pairs(true, tiles, 0, false, 0, many_resident));
        REQUIRE(!ef::server_pairs(true, tiles, (tiles - 1) / 1024, false, tiles / 2, many_resident));
        REQUIRE(ef::server_pairs(true, tiles, tiles / 1024 + 1, false, 0, many_resident) == large);
        REQUIRE(ef::server_pairs(true, tiles, tiles, true, 0, many_resident) == large);
        REQUIRE(ef::server_pairs(true, tiles, 0, false, tiles / 2 + 1, many_resident) == large);
    }
    // what a block beyond the one-pass limit parks: as many whole tiles as the limit are kept, one less where that makes an
    // even number of parked ones; without a limit none.  A parked tile's group ends in a parked tile (it is what the
    // others wait for), and all tiles of a group name the same one.
    for (int whole = 1; whole <= 130; ++whole)
        for (int keep : {0, 1, 2, 3, 7, 16, 64, 100, 129, 130, 1000}) {
            const int64_t first = 1000003;
            const int parked = ef::parked_tiles(whole, keep), kept = whole - parked;
            REQUIRE(parked >= 0 && kept >= 0 && kept <= keep);
            REQUIRE(kept == 0 || (parked % 2 == 0 && kept >= (keep < whole ? keep : whole) - 1));
            REQUIRE(kept > 0 || keep <= 1);
            REQUIRE(ef::first_kept(first, whole, keep) == first + parked);
            for (int group : {2, 3, 5, 16, 256})
                for (int64_t t = first; t < first + parked; ++t) {
                    const int64_t g0 = ef::group_first(t, first, group), g1 = ef::group_last(g0, group, first + parked);
                    REQUIRE(g0 >= first && g0 <= t && t <= g1 && g1 < g0 + group);
                    REQUIRE(g1 < first + parked);
                    REQUIRE(g1 == g0 + group - 1 || g1 + 1 == first + parked);
                    REQUIRE((g0 - first) % group == 0 && ef::group_first(g1, first, group) == g0);
                }
        }

    // an entry gives back what was put into it, to its own call alone
    for (unsigned call : {1u, 2u, 77u, (1u << 20) - 1u, 1u << 20, 0xfffffffeu, 0xffffffffu})
        for (int set : {0, 1, 63, 64})
            for (int32_t tile : {0, 1, 65535, 0x7fffffff})
                for (unsigned long long flags : {0ull, ef::PARKED_BOTH, ef::PARKED_FORMS, ef::PARKED_BOTH | ef::PARKED_FORMS})
                    for (int slot : {0, 1}) {
                        const unsigned long long e = ef::parked_entry(call, set, tile, slot, flags);
                        REQUIRE(ef::parked_in(e, call) && !ef::parked_in(e, call + 1u) && !ef::parked_in(e, call - 1u));
                        REQUIRE(ef::parked_set(e) == set && ef::parked_tile(e) == tile && ef::parked_slot(e) == slot);
                        REQUIRE((e & (ef::PARKED_BOTH | ef::PARKED_FORMS)) == flags && !ef::parked_in(0ull, call));
                    }
    // what an earlier call left in the place is neither taken nor ends the search; one that does not come ends it with 0
    {
        const unsigned long long old = ef::parked_entry(6, 0, 1, 0, 0), mine = ef::parked_entry(7, 0, 2, 1, ef::PARKED_FORMS);
        int looks = 0, rests = 0;
        const auto rest = [&] { ++rests; };
        REQUIRE(ef::await_parked([&] { return ++looks < 5 ? old : mine; }, rest, 7, 100) == mine && looks == 5 && rests == 4);
        REQUIRE(ef::await_parked([&] { return old; }, rest, 7, 100) == 0ull && rests == 104);
    }
    std::puts("layout rules ok");
    return 0;
}
