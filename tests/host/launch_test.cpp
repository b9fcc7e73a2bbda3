// Host test of the launch arithmetic (ss_launch.hpp): every unit of a call is
// launched once, in order, no launch reaches 2^32 threads, and a forward's
// slots hold every tile of every view once.
#include <cstdio>
#include <vector>

#include "ss_launch.hpp"

static int failures = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("FAILED line %d: %s\n", __LINE__, #c);      \
            ++failures;                                             \
        }                                                           \
    } while (0)

int main() {
    using namespace ss;
    const int64_t edge = (int64_t)1 << 21;  // tiles x 8 blocks x 256 threads = 2^32
    for (int64_t threads : {(int64_t)256 * 8, (int64_t)256 * 16, (int64_t)256})
        for (int64_t units : {(int64_t)1, edge - 1, edge, edge + 1, ((int64_t)1 << 24) + 3, ((int64_t)1 << 31) - 1}) {
            int64_t next = 0, pieces = 0;
            in_pieces(units, threads, [&](int64_t first, int64_t count) {
                CHECK(first == next && count >= 1);
                CHECK(count * threads < (int64_t)1 << 32);
                next = first + count;
                ++pieces;
            });
            CHECK(next == units);
            if (units * threads < (int64_t)1 << 32) CHECK(pieces == 1);
        }
    // forward launches: every (view, tile) in one slot, few slots beyond
    for (int V : {1, 2, 7, 8, 9, 10, 15, 16, 17, 25, 90})
        for (int tR : {1, 2, 5})
            for (int tC : {1, 3, 8}) {
                std::vector<int> seen((size_t)V * tR * tC, 0);
                const int64_t nb = fwd_blocks(tR, tC, V);
                for (int64_t b = 0; b < nb; ++b) {
                    int v = -1, tr = -1, tc = -1;
                    if (fwd_slot((unsigned)b, V, fwd_views(V), tR, tC, v, tr, tc)) ++seen[((size_t)v * tR + tr) * tC + tc];
                }
                for (int k : seen) CHECK(k == 1);
                // whole groups, and 10/9 of the views at most, in dealing rounds of eight items
                const int64_t whole = (int64_t)(tR > 1 ? (tR + 1) / 2 * 2 : 1) * (tC > 1 ? (tC + 1) / 2 * 2 : 1) * V;
                CHECK(nb <= whole * 10 / 9 + 7 * 4 * fwd_views(V));
            }
    // and no launch reaches the limit
    struct { int tR, tC, V; } big[] = {{1, (1 << 23) + 1, 2}, {1, 1 << 23, 3}, {1, 1, (1 << 24) + 1}, {64, 64, 8191},
                                       {1, 932000, 9}, {1, (1 << 24) - 16, 1}};
    for (auto g : big) {
        int next = 0;
        CHECK(fwd_in_pieces(g.tR, g.tC, g.V, [&](int v0, int V) {
            CHECK(v0 == next && V >= 1 && fwd_blocks(g.tR, g.tC, V) * 256 < (int64_t)1 << 32);
            next = v0 + V;
        }));
        CHECK(next == g.V);
    }
    CHECK(!fwd_in_pieces(1, 1 << 24, 1, [&](int, int) { CHECK(false); }));  // one view of 2^24 slots
    if (failures == 0) std::printf("all checks passed\n");
    return failures != 0;
}
