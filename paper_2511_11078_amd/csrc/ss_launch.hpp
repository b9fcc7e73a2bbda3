// ss_launch.hpp -- host arithmetic of kernel launches (no HIP: the host tests
// compile it by itself).
#pragma once

#include <algorithm>
#include <cstdint>

namespace ss {

// HIP takes a grid of fewer than 2^32 threads per dimension; a call has up to
// 2^31 - 1 rays, and a network block evaluates 16 or 32 of them with 256
// threads.
constexpr int64_t GRID_MAX_THREADS = ((int64_t)1 << 32) - 1;

// launch(first, count) over 0 .. units - 1 in as many pieces as that takes,
// for launches of `threads` threads per unit.
template <class Launch>
void in_pieces(int64_t units, int64_t threads, Launch launch) {
    const int64_t most = GRID_MAX_THREADS / threads;
    for (int64_t first = 0; first < units; first += most) launch(first, std::min(most, units - first));
}

}  // namespace ss
