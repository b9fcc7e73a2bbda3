// Host test of the launch arithmetic (ss_launch.hpp): every unit of a call is
// launched once, in order, and no launch reaches 2^32 threads.
#include <cstdio>

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
    if (failures == 0) std::printf("all checks passed\n");
    return failures != 0;
}
