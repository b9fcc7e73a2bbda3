// ss_launch.hpp -- arithmetic of kernel launches (no HIP: the host tests
// compile it by itself; constexpr functions serve the kernels too).
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

// XCD that takes the first of eight items of dealing round e
constexpr int xcd_rotation(int e) { return e + e / 8 + e / 64; }

// Forward launches: one 256-thread block per 16x16-pixel tile and view.
// 2 x 2 tiles of up to FT_V consecutive views form an item, whose
// blocks run on one XCD (hardware block h runs on XCD h % 8) and walk
// neighbouring lines, which share coefficient lines in its L2.  The items go
// to the XCDs eight at a time, each eight rotated against the last ones:
// every XCD takes items from all over the detector and from all views, so
// that they end together.  Before, whole groups of
// tiles with all their views went to the XCDs in turn, and an XCD could get
// the detector's edge or twice another's share: 200 views of 50 x 180 pixels
// degree 2 3.65 -> 2.42 ms, degree 0 0.70 -> 0.47; 90 views of 111 x 147
// degree 1 0.349 -> 0.284; cone_256 degree 3 150 -> 143, degree 2 71.9 -> 67.3.
// Views per item 8, 16, 32: 2.42, 2.48, 2.79 and 0.284, 0.295, 0.302 ms.
// Few slots stay empty: the views are spread evenly over a group's items (with
// eight in all but the last, nine views took the slots of sixteen), and a
// detector of one row or column of tiles has groups of one (with 2 x 2, every
// second run of sixteen blocks was empty and half of the CUs went without).
constexpr int FT_V = 8;
constexpr int fwd_views(int V) {
    const int items = (V - 1) / FT_V + 1;
    return (V - 1) / items + 1;
}
constexpr int fwd_side(int tiles) { return tiles < 2 ? 1 : 2; }  // of a group
constexpr int fwd_groups(int tR, int tC) {
    return ((tR - 1) / fwd_side(tR) + 1) * ((tC - 1) / fwd_side(tC) + 1);
}
constexpr int fwd_items(int tR, int tC, int V) {
    return fwd_groups(tR, tC) * ((V - 1) / fwd_views(V) + 1);
}
constexpr int64_t fwd_blocks(int tR, int tC, int V) {
    return (int64_t)((fwd_items(tR, tC, V) + 7) / 8 * 8) * fwd_side(tR) * fwd_side(tC) * fwd_views(V);
}
// View and tile of a block; false for a padding slot.  nv = fwd_views(V),
// from the host (a division per block cost a per-pair forward of six views up
// to 3 %; so did passing all of the order, which takes the arguments beyond
// 64 bytes).
constexpr bool fwd_slot(unsigned block, int V, int nv, int tR, int tC, int &v, int &tr, int &tc) {
    const int gh = fwd_side(tR), gw = fwd_side(tC), per = gh * gw * nv, nch = (V + nv - 1) / nv;
    const int l = (int)(block / 8), e = l / per, inner = l % per;
    const int item = e * 8 + (((int)(block & 7) + xcd_rotation(e)) & 7);
    if (item >= fwd_groups(tR, tC) * nch) return false;
    const int G = item / nch, q = inner / nv;
    v = item % nch * nv + inner % nv;
    const int gC = (tC - 1) / gw + 1;
    tr = (G / gC) * gh + q / gw;
    tc = (G % gC) * gw + q % gw;
    return v < V && tr < tR && tc < tC;
}
// Views of the largest such launch that stays below the limit (0: not even
// one does).
constexpr int fwd_launch_views(int tR, int tC, int V) {
    constexpr int64_t most = GRID_MAX_THREADS / 256;
    if (fwd_blocks(tR, tC, V) <= most) return V;
    const int64_t rounds = (most / (fwd_side(tR) * fwd_side(tC) * FT_V) - 7) / fwd_groups(tR, tC);
    if (rounds > 0) return (int)(rounds * FT_V);
    for (int v = FT_V - 1; v > 0; --v)
        if (fwd_blocks(tR, tC, v) <= most) return v;
    return 0;
}
// launch(first view, count) over V views; false if a view does not fit.
template <class Launch>
bool fwd_in_pieces(int tR, int tC, int V, Launch launch) {
    const int most = fwd_launch_views(tR, tC, V);
    for (int64_t first = 0; most > 0 && first < V; first += most)
        launch((int)first, (int)std::min<int64_t>(most, V - first));
    return most > 0;
}

}  // namespace ss
