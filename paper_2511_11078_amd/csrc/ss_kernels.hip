// ss_kernels.hip -- gfx950 kernels of the spline x-ray transform.
//
//   pad_volume_zfast_kernel, pad_volume_kernel + project_kernel
//                       forward model, one line per lane or per four lanes (quadrature form)
//   backproject_cells_kernel + cells_to_coeffs_kernel
//                       transpose: knot-cell gather, then coefficient gather (atomic-free)
//   footprint_kernel    P phi(w, x) for arbitrary pairs (diagnostics)
//   dot / axpy / xpay / ratio kernels for the least-squares loop
//
// The network form lives in ss_mlp.hip and shares the line set-up, block
// order and detector mapping of ss_math.hpp and ss_traverse.hpp.
#include "ss_kernels.hpp"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace ss {

// Zero-padded copy of the coefficients for the forward walk: FWD_PAD(n)
// zero layers on every side, so that the (n+1)^3 block of every knot cell of
// the support-padded box (and of one cell beyond) is inside the copy.
__global__ void __launch_bounds__(256) pad_volume_kernel(const float *__restrict__ c, int N0, int N1, int N2, int P,
                                                         float *__restrict__ out) {
    const int S0 = N0 + 2 * P, S1 = N1 + 2 * P, S2 = N2 + 2 * P;
    const int64_t total = (int64_t)S0 * S1 * S2;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const int x = (int)(i % S0) - P;
        const int64_t r = i / S0;
        const int yy = (int)(r % S1) - P, z = (int)(r / S1) - P;
        const bool in = x >= 0 && x < N0 && yy >= 0 && yy < N1 && z >= 0 && z < N2;
        out[i] = in ? c[((int64_t)z * N1 + yy) * N0 + x] : 0.0f;
    }
}

// The same copy with z fastest (element (x, y, z) at
// ((y + P) (N0 + 2P) + x + P) (N2 + 2P) + z + P); each block transposes a
// 32 x 32 (x, z) tile of one y layer through LDS.
constexpr int PAD_T = 32;
__global__ void __launch_bounds__(256) pad_volume_zfast_kernel(const float *__restrict__ c, int N0, int N1, int N2,
                                                              int P, float *__restrict__ out) {
    __shared__ float tile[PAD_T][PAD_T + 1];
    const int Sx = N0 + 2 * P, Sz = N2 + 2 * P;
    const int nx = (Sx + PAD_T - 1) / PAD_T, nz = (Sz + PAD_T - 1) / PAD_T;
    const int yp = (int)(blockIdx.x / (nx * nz)), b = (int)(blockIdx.x % (nx * nz)), bz = b / nx, bx = b % nx;
    const int tx = threadIdx.x % PAD_T, ty = threadIdx.x / PAD_T;
    const int y = yp - P;
    for (int k = 0; k < PAD_T; k += 256 / PAD_T) {
        const int xp = bx * PAD_T + tx, zp = bz * PAD_T + ty + k, x = xp - P, z = zp - P;
        const bool in = x >= 0 && x < N0 && y >= 0 && y < N1 && z >= 0 && z < N2;
        tile[ty + k][tx] = in ? c[((int64_t)z * N1 + y) * N0 + x] : 0.0f;
    }
    __syncthreads();
    for (int k = 0; k < PAD_T; k += 256 / PAD_T) {
        const int zp = bz * PAD_T + tx, xp = bx * PAD_T + ty + k;
        if (xp < Sx && zp < Sz) out[((int64_t)yp * Sx + xp) * Sz + zp] = tile[tx][ty + k];
    }
}

// How the forward walks view e.
//
// What limits the walk beside its arithmetic is the rate of the L1 cache's
// row reads: a 16-byte read per lane costs, for each group of four lanes, one
// step per cache-line segment the four touch (loads alone, the integral
// replaced by a sum, took 146 of cone_256's 164 ms with rows along x or y,
// whatever the occupancy).  So the lanes of a wave are laid along the
// detector direction that runs best along an axis, over the copy with that
// axis fastest: z (the rows of a circular trajectory: cone_256 degree 3
// 163.5 -> 150 ms, degree 2 85.5 -> 72, degree 1 38.5 -> 29, degree 0
// 23.5 -> 12 ms), or x where that fits better (rays along z).
//
// `yorder`: which of x and y is contracted first (y: central ray within 15
// degrees of x, or between 15 and 35 degrees of y).  It has no bearing on
// speed; it fixes the order of the FP32 sums.
//
// The host evaluates it too (project_quad_walks_x): a geometry none of whose
// views fits x better, as every circular trajectory about z, makes and holds
// the z-fastest copy alone (two: 0.05 + 0.04 ms and 147 MB on cone_256; a
// degree-0 call of 16^3 15.9 and 12.5 us).
struct ViewWalk {
    bool yorder, xcopy, rows;  // rows: lanes along the detector's rows
};
template <int n>
__host__ __device__ __forceinline__ ViewWalk view_walk(const float *__restrict__ e, int kind) {
    ViewWalk vw;
    float d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = kind != 0 ? e[3 + k] - e[k] : e[k];  // cone: source -> detector centre
    const float ax = fabsf(d[0]), ay = fabsf(d[1]), az = fabsf(d[2]);
    const float hi = fmaxf(ax, ay), lo = fminf(ax, ay);
    const float s = lo / hi;                        // tan(phi)
    constexpr float T15 = 0.26794919f, T35 = 0.70020754f;
    vw.yorder = n >= 1 && az < hi && (ax >= ay ? s < T15 : (s >= T15 && s < T35));
    // squared cosines of the detector's two directions with z and x
    const float iu = 1.0f / (e[6] * e[6] + e[7] * e[7] + e[8] * e[8]);
    const float iv = 1.0f / (e[9] * e[9] + e[10] * e[10] + e[11] * e[11]);
    const float zu = e[8] * e[8] * iu, zv = e[11] * e[11] * iv, xu = e[6] * e[6] * iu, xv = e[9] * e[9] * iv;
    vw.xcopy = !vw.yorder && fmaxf(xu, xv) > fmaxf(zu, zv);
    vw.rows = vw.xcopy ? xv > xu : !(zu > zv);
    return vw;
}

// ---------------------------------------------------------------------------
// Forward, quadrature form: cell walk.  The footprint of a basis is the sum,
// over the knot cells its support spans, of the Gauss-Legendre integral of
// its (polynomial) restriction to the line inside the cell.  Walking the
// line cell by cell through the knot lattice (Amanatides-Woo stepping over
// the support-padded box) and adding, for every cell, c_q times that
// per-cell integral for each of the (n+1)^3 bases whose support covers the
// cell visits every (line, basis) pair of eq. (4) exactly once, through the
// same Gauss-Legendre terms as the slab-by-slab per-basis sum, evaluated
// with the node positions and per-axis weights shared by the (n+1)^3 bases.
// ---------------------------------------------------------------------------

// Launches of up to this many 16 x 16-pixel tiles share each line among four
// lanes (project_kernel), by degree and by the copy's size (up to
// FWD_SHARED_FLOATS, and above): all four walk the whole line, so the
// shorter the integral the sooner that costs more than it gives, and a wave of
// sixteen lines reads more cache lines per integral, which counts once the
// copy is large.  Shared and not, us, views of 1.5 N x 1.5 N pixels over N^3,
// lines 2/3 of a coefficient apart:
//   degree 0  N = 64 324 tiles 47 and 47, 504 59 and 46; 128 432 96 and 114, 576 120 and 89
//   degree 1  N = 64 216 57 and 60, 324 66 and 59; 128 288 100 and 108, 576 167 and 112
//   degree 2  N = 24 522 55 and 62, 954 86 and 74; 96 486 210 and 208, 648 252 and 191;
//             160 225 167 and 223, 450 282 and 233
//   degree 3  N = 48 525 190 and 207, 1150 382 and 371; 96 486 373 and 410, 648 463 and 396;
//             160 225 324 and 395, 450 500 and 427; 256 1152 1742 and 1428
// Lines further apart than FWD_SPARSE coefficients have few cache lines in
// common within a wave of 64 either: what overlaps is the four lanes'
// consecutive cells, and the launch may be larger (degree 3, 256^3, 16 views
// of 96 x 96 pixels 3.4 apart, 576 tiles 1.14 and 2.37 ms; 384^3, one view of
// 352 x 352 1.4 apart 1.08 and 1.24, 4 views of 256 x 256 1.9 apart 2.40 and
// 2.29; 256^3, 4 views of 256 x 256 1.27 apart 1.48 and 1.17).
constexpr int64_t FWD_SHARED_TILES[4][2] = {{330, 490}, {320, 320}, {560, 440}, {640, 440}};
constexpr int64_t FWD_SHARED_FLOATS = (int64_t)1 << 21;
constexpr int64_t FWD_SPARSE_TILES[4] = {512, 320, 768, 1536};
constexpr float FWD_SPARSE = 1.3f;
// Copies of up to this many floats (128 MiB) are walked in waves of 8 x 8
// pixels instead of 16 x 4 at degrees 2 and 3.  Square waves idle less where
// lines leave the volume (16 x 4 against 8 x 8: 128^3 with 192^2 pixels
// degree 3 12.5 and 11.5 ms, degree 2 5.6 and 5.2; 180 x 180 x 50 with 50 x
// 180 pixels degree 2 3.9 and 3.6; 256^3 with 384^2 150.7 and 150.8);
// long ones read fewer cache lines, which counts where the copy is large
// (384^3 53.7 and 54.1, 512^3 127.4 and 128.9) or the integral short (cone_256
// degree 1 29.4 and 30.3, degree 0 12.0 and 12.4).
constexpr int64_t FWD_SQUARE_FLOATS = (int64_t)1 << 25;
// Largest padded copy (floats, 1 GiB) that is kept in both orders, so that
// one launch walks every view.
constexpr int64_t FWD_BOTH_FLOATS = (int64_t)1 << 28;

// pointers that keep their address space through an empty asm
typedef const __attribute__((address_space(1))) char *GlobalBytes;
typedef const __attribute__((address_space(1))) float *GlobalFloats;

// v_min_f64 as it stands: fmin() quiets both operands first, two more FP64
// instructions each (no NaN reaches the walk)
__device__ __forceinline__ double min64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// One (line, cell) unit: half the integral of c's restriction to the cell
// over xi in [-1, 1], from the cell's coefficient block.  lc: local
// coordinates of the chord's mid-point, dl: their step to its end.
template <int n>
__device__ __forceinline__ float cell_integral(const float (&cb)[n + 1][n + 1][n + 1], const float lc[3],
                                               const float dl[3]) {
    using Rule = GLRule<Degree<n>::m>;
    constexpr int NB = n + 1;
    float seg = 0.0f;
#pragma unroll
    for (int l = 0; l < Rule::m; ++l) {
        const float xi = Rule::x(l);
        float w1[NB], w2[NB], w3[NB];
        cell_weights<n>(xi == 0.0f ? lc[0] : fmaf(dl[0], xi, lc[0]), w1);
        cell_weights<n>(xi == 0.0f ? lc[1] : fmaf(dl[1], xi, lc[1]), w2);
        cell_weights<n>(xi == 0.0f ? lc[2] : fmaf(dl[2], xi, lc[2]), w3);
        float f = 0.0f;
#pragma unroll
        for (int a3 = 0; a3 < NB; ++a3) {
            float g = 0.0f;
#pragma unroll
            for (int a2 = 0; a2 < NB; ++a2) {
                float r = 0.0f;
#pragma unroll
                for (int a1 = 0; a1 < NB; ++a1) r = fmaf(w1[a1], cb[a3][a2][a1], r);
                g = fmaf(w2[a2], r, g);
            }
            f = fmaf(w3[a3], g, f);
        }
        seg = fmaf(0.5f * Rule::w(l), f, seg);
    }
    return seg;
}

// value of lane (quad base + P) of each quad
template <int P>
__device__ __forceinline__ float quad_lane(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), P * 0x55, 0xf, 0xf, true));
}

// `which` = 2: every view, each in the copy it walks (view_walk; both copies
// are there, or, cx null, the z-fastest one alone, which then serves a view
// whose two cosines tie but for rounding as well).  0 and 1: only the views of the z- and of the x-fastest copy
// (blocks of the others return at once), for a scratch that holds one copy
// at a time.
//
// What bounds it at degree 3: VALU issue (the cell integral's about 630
// instructions; with every load at one address the kernel took 137 ms on
// cone_256) and the L1 reads (view_walk).  The walk around the integral is
// kept short: cell indices are carried as the FP64 numbers and the byte
// offset the cell needs, an axis that reaches its plane advances under its
// own mask (ties advance together instead of by cells of no length), and a
// row's address is a scalar base plus that one 32-bit offset (WIDE: copies
// above 4 GiB, 64-bit).  727 -> 675 VALU instructions per (line, cell).
//
// LPL lanes share a line: LPL = 4 lets a launch of few lines fill the chip
// (small_parallel_32: 450 -> 115 us for 288 tiles).  Each of the four walks
// all of the line's cells, integrates every fourth one, and all four add the
// terms in the line's order, so that the sum is the same bit for bit.
template <int n, int LPL, bool WIDE>
__global__ void __launch_bounds__(256, n == 3 ? 3 : 4) project_kernel(const float *__restrict__ cz,
                                                                     const float *__restrict__ cx, int N0, int N1,
                                                                     int N2, const float *__restrict__ geom, int kind,
                                                                     int V, int R, int C, float *__restrict__ y,
                                                                     int which, int nv) {
    constexpr int NB = n + 1;
    constexpr double h = (double)Degree<n>::h;
    constexpr double kap = (double)Degree<n>::kap;
    constexpr int qoff = CellBasis<n>::qoff;
    using Off = typename std::conditional<WIDE, uint64_t, uint32_t>::type;
    const int tR = (R + 15) / 16, tC = (C + 15) / 16;
    int v, tr, tc_, part = 0;
    if constexpr (LPL == 1) {
        if (!fwd_block_tile(V, nv, tR, tC, v, tr, tc_)) return;  // padding slot
    } else {
        // four blocks per 16 x 16-pixel tile, tiles innermost: a launch this
        // small spreads evenly over the chip
        const int t = blockIdx.x / LPL;
        part = blockIdx.x % LPL;
        tc_ = t % tC;
        tr = (t / tC) % tR;
        v = t / (tC * tR);
    }
    if (v >= V) return;
    ViewWalk vw = view_walk<n>(geom + 12 * v, kind);
    if (!cx) vw.xcopy = false;
    if (which != 2 && vw.xcopy != (which != 0)) return;  // the other copy's view
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane & (LPL - 1);
    int j, i;
    if constexpr (LPL == 1) {
        // a wave takes 16 x 4 pixels, consecutive lanes along the long side,
        // or 8 x 8 (FWD_SQUARE_FLOATS)
        const bool square = n >= 2 && !WIDE &&
                            (int64_t)(N0 + 2 * FWD_PAD(n)) * (N1 + 2 * FWD_PAD(n)) * (N2 + 2 * FWD_PAD(n)) <=
                                FWD_SQUARE_FLOATS;
        const int along = square ? (wave >> 1) * 8 + (lane & 7) : lane & 15;
        const int across = square ? (wave & 1) * 8 + (lane >> 3) : wave * 4 + (lane >> 4);
        j = tr * 16 + (vw.rows ? along : across);
        i = tc_ * 16 + (vw.rows ? across : along);
    } else {
        j = tr * 16 + (part >> 1) * 8 + (wave >> 1) * 4 + (lane >> 4);
        i = tc_ * 16 + (part & 1) * 8 + (wave & 1) * 4 + ((lane >> 2) & 3);
    }
    if (j >= R || i >= C) return;
    // the walk runs in the order of the contractions: (x, y, z), or (y, x, z)
    const int N[3] = {vw.yorder ? N1 : N0, vw.yorder ? N0 : N1, N2};
    const double centre[3] = {0.0, 0.0, 0.0};
    LineD L = make_line(geom + 12 * v, kind, R, C, j, i, centre);
    if (vw.yorder) {
        const double a0 = L.a[0], w0 = L.w[0];
        L.a[0] = L.a[1]; L.a[1] = a0;
        L.w[0] = L.w[1]; L.w[1] = w0;
    }
    float acc = 0.0f;
    if (L.ok) {
        // index coordinates z = x - o, o = -(N - 1)/2
        double z0[3], t0 = -1e300, t1 = 1e300;
        bool hit = true;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            z0[k] = L.a[k] + 0.5 * (double)(N[k] - 1);
            const double lo = -h, hi = (double)(N[k] - 1) + h;
            if (L.w[k] == 0.0) {
                if (!(z0[k] > lo && z0[k] < hi)) hit = false;
                // degree 0: the support of beta^0 is open, so a line lying in
                // a face plane between two voxels meets neither
                if (n == 0 && z0[k] - kap == floor(z0[k] - kap)) hit = false;
            } else {
                const double ta = (lo - z0[k]) / L.w[k], tb = (hi - z0[k]) / L.w[k];
                t0 = fmax(t0, fmin(ta, tb));
                t1 = fmin(t1, fmax(ta, tb));
            }
        }
        if (hit && t0 < t1) {
            // zero-padded copy of the coefficients (FWD_PAD(n) layers per
            // side), and its strides in bytes along the walk's axes
            constexpr int P = FWD_PAD(n);
            const int64_t Sx = N0 + 2 * P, Sy = N1 + 2 * P, Sz = N2 + 2 * P;
            const int64_t strx = vw.xcopy ? 4 : 4 * Sz, stry = vw.xcopy ? 4 * Sx : 4 * Sz * Sx;
            const int64_t str[3] = {vw.yorder ? stry : strx, vw.yorder ? strx : stry, vw.xcopy ? 4 * Sx * Sy : 4};
            const Off last = (Off)(str[0] * (N[0] + 2 * P - NB) + str[1] * (N[1] + 2 * P - NB) +
                                   str[2] * (N[2] + 2 * P - NB));
            // DDA state per axis: parameter of the next knot plane and its
            // step, the cell's lower knot plane and its step, and the byte
            // offset of the cell's coefficient block and its steps
            double tmax[3], tdel[3], md[3], ms[3], wh[3];
            Off os[3], off = 0;
            {
                int m[3];
                // a point just past the entry (the entry lies on a knot plane)
                const double tm0 = t0 + fmin(1e-6, 0.5 * (t1 - t0));
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double zs = fma(tm0, L.w[k], z0[k]) - kap;
                    m[k] = (int)floor(fmin(fmax(zs, -8.0), (double)N[k] + 8.0));
                    md[k] = (double)m[k] + kap;
                    wh[k] = 0.5 * L.w[k];
                    if (L.w[k] > 0.0) {
                        ms[k] = 1.0;
                        os[k] = (Off)str[k];
                        tdel[k] = 1.0 / L.w[k];
                        tmax[k] = ((double)(m[k] + 1) + kap - z0[k]) / L.w[k];
                    } else if (L.w[k] < 0.0) {
                        ms[k] = -1.0;
                        os[k] = (Off)-str[k];
                        tdel[k] = -1.0 / L.w[k];
                        tmax[k] = ((double)m[k] + kap - z0[k]) / L.w[k];
                    } else {
                        ms[k] = 0.0;
                        os[k] = 0;
                        tdel[k] = 0.0;
                        tmax[k] = 1e300;
                    }
                    off += (Off)((m[k] + qoff + P) * str[k]);
                }
            }
            // to the next knot plane of whichever axes reach theirs first:
            // the walk ends after at most sum_k (N_k + 2h + 2) steps
            double tc = t0;
            auto advance = [&](double tn) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (tmax[k] <= tn) {
                        asm volatile("");  // under a mask, not by selects
                        tmax[k] += tdel[k];
                        md[k] += ms[k];
                        off += os[k];
                    }
            };
            // the walk over a copy whose fastest axis is the contractions'
            // third (z) or, XC, their first (x)
            auto walk = [&](auto xc) {
                constexpr bool XC = decltype(xc)::value;
                // first element of each row of a block, in scalar registers
                // (kept apart by the empty asm: one base and sixteen 64-bit
                // vector additions per cell otherwise)
                GlobalBytes rowp[NB][NB];
#pragma unroll
                for (int r1 = 0; r1 < NB; ++r1)
#pragma unroll
                    for (int r0 = 0; r0 < NB; ++r0) {
                        rowp[r1][r0] = XC ? (GlobalBytes)cx + (r1 * str[2] + r0 * str[1])
                                          : (GlobalBytes)cz + (r1 * str[1] + r0 * str[0]);
                        asm("" : "+s"(rowp[r1][r0]));
                    }
                // the unit between parameters ta and tb of the cell with
                // lower knot planes cm and block offset o; returns its
                // term's two factors
                auto unit = [&](double ta, double tb, const double cm[3], Off o, float &len) {
                    // every cell of the walk lies in the support-padded box
                    // or one cell beyond it, so its block is inside the copy;
                    // the clamp only guards the address
                    const Off ob = o < last ? o : last;
                    float cb[NB][NB][NB];
#pragma unroll
                    for (int r1 = 0; r1 < NB; ++r1)
#pragma unroll
                        for (int r0 = 0; r0 < NB; ++r0) {
                            const auto row = (GlobalFloats)(rowp[r1][r0] + ob);
#pragma unroll
                            for (int q = 0; q < NB; ++q) (XC ? cb[r1][r0][q] : cb[q][r1][r0]) = row[q];
                        }
                    // all loads first: spread over the integral they would
                    // each be waited for (184 against 163 ms)
                    __builtin_amdgcn_sched_barrier(0);
                    // mid-point and half-length in the line's parameter, the
                    // factor 1/2 carried by wh (and in cell_integral)
                    const double sum = ta + tb, dif = tb - ta;
                    float lc[3], dl[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        lc[k] = (float)(fma(sum, wh[k], z0[k]) - cm[k]);
                        dl[k] = (float)(dif * wh[k]);
                    }
                    len = (float)dif;
                    return cell_integral<n>(cb, lc, dl);
                };
                if constexpr (LPL == 1) {
                    while (tc < t1) {
                        const double tn = min64(min64(tmax[0], tmax[1]), tmax[2]), te = min64(tn, t1);
                        if (te > tc) {
                            float len;
                            const float seg = unit(tc, te, md, off, len);
                            acc = fmaf(len, seg, acc);
                            tc = te;
                        }
                        advance(tn);
                    }
                } else {
                    while (tc < t1) {
                        // the next four units of the line, one for each lane
                        int got = 0;
                        double ua = 0.0, ub = 0.0, um[3] = {0.0, 0.0, 0.0};
                        Off uo = 0;
                        while (tc < t1 && got < LPL) {
                            const double tn = min64(min64(tmax[0], tmax[1]), tmax[2]), te = min64(tn, t1);
                            if (te > tc) {
                                if (got == sub) {
                                    ua = tc;
                                    ub = te;
                                    um[0] = md[0]; um[1] = md[1]; um[2] = md[2];
                                    uo = off;
                                }
                                ++got;
                                tc = te;
                            }
                            advance(tn);
                        }
                        float len = 0.0f, seg = 0.0f;
                        if (sub < got) seg = unit(ua, ub, um, uo, len);
                        acc = got > 0 ? fmaf(quad_lane<0>(len), quad_lane<0>(seg), acc) : acc;
                        acc = got > 1 ? fmaf(quad_lane<1>(len), quad_lane<1>(seg), acc) : acc;
                        acc = got > 2 ? fmaf(quad_lane<2>(len), quad_lane<2>(seg), acc) : acc;
                        acc = got > 3 ? fmaf(quad_lane<3>(len), quad_lane<3>(seg), acc) : acc;
                    }
                }
            };
            if (vw.xcopy) walk(std::true_type{});
            else walk(std::false_type{});
        }
    }
    if (sub == 0) y[((int64_t)v * R + j) * C + i] = acc;
}

// ---------------------------------------------------------------------------
// Adjoint, quadrature form: cell gather, two passes, no atomics.
//
// The transpose of the forward cell walk: line m adds y_m times the
// Gauss-Legendre integral, over its chord through knot cell K, of the
// restriction of basis q to the line, for each of the (n+1)^3 bases q whose
// support covers K.  Pass 1 gives every knot cell to one thread, which
// gathers, over all views, the lines of the pixels whose centres fall in the
// detector shadow of its cell, accumulates the centred moments of their
// chords (integrate_hit) and at the end maps them to the (n+1)^3 per-basis
// integrals (entry a = q - K - qoff per axis of cell K), which the block sums
// per coefficient over its cells.  Pass 2 gives every coefficient to one
// thread, which adds its parts of the blocks that hold cells of its support.
// Every (line, basis) pair of eq. (4) is evaluated through the same per-cell
// Gauss-Legendre terms as the forward, each output has a single writer, and
// the summation order is fixed.
//
// Pass 1 blocks own GX x GY x GZ bricks of cells and take the views in
// batches: as many consecutive views as fit half of the LDS line table (a
// few hundred lines, up to 8 views; a view whose shadow is larger
// than that is taken alone, in segments, each like a batch).  Per batch the
// block
//   - fills the half with the lines of each view's pixel rectangle (FP64
//     set-up, anchor re-based at the brick centre), all threads taking part
//     whatever the view,
//   - and every thread computes, view by view, the pixel rectangle of its
//     own cell's shadow (about 95 % of those lines hit the cell) and appends
//     it to its queue as one 32-bit run (first table entry, columns, rows).
// A thread's shadow is bounded around its projected cell centre: with
// den = 1 at the source plane's parallel through the detector, the position
// moves by at most F / (den - hn) pixels over the cell, F = half the sum
// over axes of |du_k - (nu/den) nm_k| taken at the ends of nu/den over the
// brick, hn half the sum of |nm_k| (0.5 % above the exact bound, no corner
// table, no LDS reads).  The views' rectangles and per-brick constants are
// computed by 64 threads for 64 views at a time.  Integration drains the
// queues: before a half is refilled, each wave runs as many rounds as its
// lane with the most entries in that half needs, and lanes with fewer take
// entries of the other half in the same rounds, so that the lanes of a wave,
// whose candidate counts differ view by view, stay busy.  (Segments that
// emptied the queues each time took, at 60^3 with 24 parallel views of 4 x 4
// pixels per coefficient, 1.20 instead of 0.90 ms at degree 0, 1.59 and 1.07,
// 3.31 and 2.04, 5.60 and 3.69 at degree 3; only where a cell may have more
// than 60 pixels in a row or column are they still.)
//
// What bounds it: VALU issue, 2.07 hits of about 440 instructions per (cell,
// view) plus the set-up, at 0.36 wave instructions per SIMD per cycle (degree
// 3; independent FMAs reach 0.41).  With a corner table, a barrier and a
// partly filled line set-up per view instead of per batch, and a queue of
// single entries, cone_256 took 187.5 ms at degree 3 and 70.9 ms at degree 0
// (1.43e11 and 3.79e10 VALU instructions); with the batches and the plain slab
// test for tables without axis-parallel lines 153 and 46.1 ms (1.27e11 and
// 2.3e10, half the scalar ones), with the bricks dealt to the XCDs (xcd_remap)
// 143 and 41.6; bit for bit the same sums.
//
// The table between the passes holds, per block, the FP64 parts of the
// coefficients whose support meets its cells (11 x 11 x 7 for 8 x 8 x 4 cells
// at degree 3: 6.8 KB, where the entries of the cells themselves take 64 KB;
// 512^3, 32 views of 768 x 768: 35.6 -> 3.7 GB of table, 134 -> 127 ms;
// cone_256 4.5 -> 0.5 GB, 156.6 -> 155.1 ms; degrees 0 and 1 unchanged).
// Volumes whose table would exceed the context's scratch are processed in
// overlapping z-chunks of cell layers: a chunk of L layers finalises L - n
// coefficient layers.
// ---------------------------------------------------------------------------
constexpr int GX = 8, GY = 8, GZ = 4;
constexpr int RUN_MAX = 64;           // most columns and rows of a run (6 bits each)
constexpr int BV_CHUNK = 64;          // views whose brick constants are kept in LDS
struct BrickViews {
    float nc[BV_CHUNK], nr[BV_CHUNK], dn[BV_CHUNK];  // centre's numerators and denominator
    float fc[BV_CHUNK], fr[BV_CHUNK];                // F of the columns and rows
    int i0[BV_CHUNK], j0[BV_CHUNK], w[BV_CHUNK], h[BV_CHUNK];  // the brick's pixel rectangle
    int own[BV_CHUNK];  // its pixels; more than half the line table holds if the view goes alone, in segments: by one,
                        // or by two if a cell may have more pixels than fit a run
};
// Line table (two halves) and occupancy per degree: the cubic kernel's
// registers allow three waves per SIMD, so its table takes what LDS leaves
// for three blocks per CU beside the queues, counting 160 KiB in 2 KiB
// units; lower degrees fit four waves and a smaller table.
// SHARED: blocks of 64 cells, a quarter (4 x 4 x 4) of a brick, whose (n+1)^3
// moments are divided among n + 1 waves by the power of the third
// coordinate; for launches of few bricks.  Anchors and cells stay relative to
// the brick's centre and every moment is the same chain of FMAs, so the sums
// are the same bit for bit.
template <int n, bool SHARED> struct CellGather {
    static constexpr int threads = SHARED ? 64 * (n + 1) : 256;
    static constexpr int sx = SHARED ? 4 : GX, sy = SHARED ? 4 : GY;  // cells of a block (x GZ)
    static constexpr int waves = n == 3 && !SHARED ? 3 : 4;  // waves per SIMD: blocks per CU
    static constexpr int lds = (160 * 1024 / waves) / 2048 * 2048;
    static constexpr int batch = SHARED ? 4 : 8;             // views per batch: runs per thread and table half
    static constexpr int fixed = 2 * batch * threads * 4 + (int)sizeof(BrickViews) + 64;
    static constexpr int half = SHARED ? 256 : std::min((lds - fixed) / 40 / 2 / 16 * 16, 480);  // lines per half (40 bytes each)
    // coefficients whose support meets a block's cells, and that count made even
    static constexpr int coeffs = (sx + n) * (sy + n) * (GZ + n), record = (coeffs + 1) / 2 * 2;
    using Part = std::conditional_t<n == 0, float, double>;  // a coefficient's part (degree 0: one FP32 entry)
    // wave priority while a block sets up a batch (0: the default throughout)
    static constexpr int setup_prio = n == 0 ? 0 : 2;
    static_assert(2 * half <= 1024, "a run's first entry has 10 bits");
};
// Launches of up to this many bricks, one per CU, share each cell's moments
// (SHARED) at degrees 2 and 3: 32 views, degree 3, 225 bricks 164 -> 110 us,
// 396 bricks 176 and 170, 637 bricks 208 and 234; degree 2, 225 bricks
// 79 -> 72; degree 1 gains nothing (69 and 71).
constexpr int SHARED_BRICKS = 256;
constexpr float PIX_MARGIN = 1.0e-3f;           // pixels; covers FP32 rounding of the shadow bounds

typedef float f32x2 __attribute__((ext_vector_type(2)));

struct __attribute__((aligned(8))) CellRay {  // 40 bytes
    float a[3];      // point of the line nearest the brick centre, relative to it
    float iw[3];     // 1 / w_k; 0 marks an axis the line is parallel to
    float w[3];      // unit direction
    float y;         // sinogram value
};

// Returns whether the line is parallel to an axis.
__device__ __forceinline__ bool fill_cellray(CellRay &rec, const float *__restrict__ e, int kind, int R, int C, int j,
                                             int i, const double centre[3], float yval) {
    const LineD L = make_line(e, kind, R, C, j, i, centre);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // a degenerate line is put far outside every cell, parallel to all axes
        const float wk = L.ok ? (float)L.w[k] : 0.0f;
        rec.a[k] = L.ok ? (float)(L.a[k] - centre[k]) : 1.0e30f;
        rec.w[k] = wk;
        rec.iw[k] = wk != 0.0f ? __builtin_amdgcn_rcpf(wk) : 0.0f;
    }
    rec.y = L.ok ? yval : 0.0f;
    return rec.iw[0] == 0.0f || rec.iw[1] == 0.0f || rec.iw[2] == 0.0f;
}

// Chord [t0, t1] of a line through the cell [lo, lo + 1]^3 (coordinates
// relative to the brick centre).  A line parallel to a knot plane belongs to
// the cell above it when it lies in the plane (the forward walk's choice);
// for degree 0 the support is open and such a line meets neither cell.
// Written without branches (selects only), so that the lanes of a wave never
// split on a parallel axis.  `flat` (uniform): whether any line of the table
// has one; without, the plain slab test gives the same values in 26 instead
// of 50 instructions.
template <int n>
__device__ __forceinline__ bool cell_chord(const CellRay &r, const float lo[3], bool flat, float &t0, float &t1) {
    if (!flat) {
        float a[3], b[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float ta = (lo[k] - r.a[k]) * r.iw[k], tb = (lo[k] + 1.0f - r.a[k]) * r.iw[k];
            a[k] = fminf(ta, tb);
            b[k] = fmaxf(ta, tb);
        }
        t0 = fmaxf(fmaxf(a[0], a[1]), a[2]);
        t1 = fminf(fminf(b[0], b[1]), b[2]);
        return t0 < t1;
    }
    bool in = true;
    t0 = -3.0e38f;
    t1 = 3.0e38f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const bool par = r.iw[k] == 0.0f;
        const bool inside = (n == 0 ? lo[k] < r.a[k] : lo[k] <= r.a[k]) & (r.a[k] < lo[k] + 1.0f);
        const float ta = (lo[k] - r.a[k]) * r.iw[k], tb = (lo[k] + 1.0f - r.a[k]) * r.iw[k];
        in = in & (inside | !par);
        t0 = par ? t0 : fmaxf(t0, fminf(ta, tb));
        t1 = par ? t1 : fminf(t1, fmaxf(ta, tb));
    }
    return in & (t0 < t1);
}

// Add one line's chord through the cell to the cell's moments: at the m
// Gauss-Legendre nodes of the chord, y * weight * u1^p1 u2^p2 u3^p3 for the
// centred cell coordinates u = t - 1/2.
// SHARED: only the moments of u3^q3 (q3 uniform), acc[p2 * (n+1) + p1].
template <int n, bool SHARED>
__device__ __forceinline__ void integrate_hit(const CellRay &r, const float lo[3], bool flat, int q3, float acc[]) {
    using Rule = GLRule<Degree<n>::m>;
    constexpr int NB = n + 1;
    float t0, t1;
    if (!cell_chord<n>(r, lo, flat, t0, t1)) return;  // a candidate whose line misses the cell
    const float mid = 0.5f * (t0 + t1), half = 0.5f * (t1 - t0);
    float uc[3], du[3];  // centred cell coordinate at mid, and its step
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        uc[q] = fmaf(mid, r.w[q], r.a[q]) - (lo[q] + 0.5f);
        du[q] = half * r.w[q];
    }
    const float sc = half * r.y;
#pragma unroll
    for (int l = 0; l < Rule::m; ++l) {
        const float xi = Rule::x(l);
        // powers u^p of the three centred coordinates (p >= 1)
        float P1[NB], P2[NB], P3[NB];
        P1[0] = Rule::w(l) * sc;  // axis 1 carries the quadrature weight
        P2[0] = 1.0f;
        P3[0] = 1.0f;
        const float u1 = xi == 0.0f ? uc[0] : fmaf(du[0], xi, uc[0]), u2 = xi == 0.0f ? uc[1] : fmaf(du[1], xi, uc[1]),
                    u3 = xi == 0.0f ? uc[2] : fmaf(du[2], xi, uc[2]);
#pragma unroll
        for (int p = 1; p <= n; ++p) {
            P1[p] = P1[p - 1] * u1;
            P2[p] = p == 1 ? u2 : P2[p - 1] * u2;
            P3[p] = p == 1 ? u3 : P3[p - 1] * u3;
        }
        if constexpr (SHARED) {
            // u3^q3 through the same products (factors of 1 are exact)
            const float t3 = (q3 >= 2 ? u3 * u3 : 1.0f) * ((q3 & 1) ? u3 : 1.0f);
            if (q3 == 0) {
                // the last product of each power fused with its sum, as
                // a + P1[p1] is below
                acc[0] = fmaf(Rule::w(l), sc, acc[0]);
#pragma unroll
                for (int p1 = 1; p1 < NB; ++p1) acc[p1] = fmaf(P1[p1 - 1], u1, acc[p1]);
            } else {
#pragma unroll
                for (int p1 = 0; p1 < NB; ++p1) acc[p1] = fmaf(t3, P1[p1], acc[p1]);
            }
#pragma unroll
            for (int p2 = 1; p2 < NB; ++p2) {
                const float z = t3 * P2[p2];
#pragma unroll
                for (int p1 = 0; p1 < NB; ++p1) acc[p2 * NB + p1] = fmaf(z, P1[p1], acc[p2 * NB + p1]);
            }
            continue;
        }
#pragma unroll
        for (int p3 = 0; p3 < NB; ++p3)
#pragma unroll
            for (int p2 = 0; p2 < NB; ++p2) {
                // z = u2^p2 u3^p3 (no product where either power is zero)
                const float z = p3 == 0 ? P2[p2] : (p2 == 0 ? P3[p3] : P3[p3] * P2[p2]);
#pragma unroll
                for (int p1 = 0; p1 < NB; ++p1) {
                    float &a = acc[(p3 * NB + p2) * NB + p1];
                    a = (p2 == 0 && p3 == 0) ? a + P1[p1] : fmaf(z, P1[p1], a);
                }
            }
    }
}

// Pixels whose centre lies in the continuous detector rectangle
// [cmin, cmax] x [rmin, rmax] (pixel units), clamped to the detector;
// PIX_MARGIN absorbs the FP32 rounding of the bounds.
__device__ __forceinline__ void pixel_rect(float cmin, float cmax, float rmin, float rmax, int R, int C, int &i0,
                                           int &i1, int &j0, int &j1) {
    // clamped in FP32 before converting
    const float fi0 = fmaxf(ceilf(cmin - PIX_MARGIN), 0.0f), fi1 = fminf(floorf(cmax + PIX_MARGIN), (float)(C - 1));
    const float fj0 = fmaxf(ceilf(rmin - PIX_MARGIN), 0.0f), fj1 = fminf(floorf(rmax + PIX_MARGIN), (float)(R - 1));
    if (fi0 <= fi1 && fj0 <= fj1) {
        i0 = (int)fi0; i1 = (int)fi1; j0 = (int)fj0; j1 = (int)fj1;
    } else {
        i0 = 0; i1 = -1; j0 = 0; j1 = -1;
    }
}

// One view's constants for the brick centred at `centre`: the numerators and
// the denominator of the centre's projection (FP64 differences), the brick's
// pixel rectangle from its eight projected corners, and the shadow
// half-widths F of its cells.  A corner on or behind the source plane has no
// bounded shadow: the whole detector, and unbounded F.
// The cells are [x0, x0 + sx] x [y0, y0 + sy] of the brick's GX x GY (all of GZ).
__device__ __forceinline__ void brick_view(const ViewProj &P, const double centre[3], int x0, int sx, int y0, int sy,
                                           int R, int C, int half, BrickViews &B, int s) {
    const float oc = 0.5f * (float)(C - 1) + P.gac_f, orow = 0.5f * (float)(R - 1) + P.gar_f;
    const double *c = centre;
    const float nc = (float)(fma(c[2], P.du_s[2], fma(c[1], P.du_s[1], c[0] * P.du_s[0])) - P.odu);
    const float nr = (float)(fma(c[2], P.dv_s[2], fma(c[1], P.dv_s[1], c[0] * P.dv_s[0])) - P.odv);
    const float dn = P.kind == 0 ? 1.0f
                     : (float)((fma(c[2], P.nrm[2], fma(c[1], P.nrm[1], c[0] * P.nrm[0])) - P.onm) / P.plane);
    bool bad = false;
    float gmin = 3.0e38f, gmax = -3.0e38f, hmin = 3.0e38f, hmax = -3.0e38f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float d[3] = {(float)(x0 + ((k & 1) ? sx : 0)) - 0.5f * GX, (float)(y0 + ((k & 2) ? sy : 0)) - 0.5f * GY,
                            (k & 4) ? 0.5f * GZ : -0.5f * GZ};
        const float den = fmaf(d[2], P.nmp_f[2], fmaf(d[1], P.nmp_f[1], fmaf(d[0], P.nmp_f[0], dn)));
        bad = bad || !(den > 0.0f);
        const float lam = __builtin_amdgcn_rcpf(den);
        const float g = lam * fmaf(d[2], P.du_f[2], fmaf(d[1], P.du_f[1], fmaf(d[0], P.du_f[0], nc)));
        const float h = lam * fmaf(d[2], P.dv_f[2], fmaf(d[1], P.dv_f[1], fmaf(d[0], P.dv_f[0], nr)));
        gmin = fminf(gmin, g); gmax = fmaxf(gmax, g);
        hmin = fminf(hmin, h); hmax = fmaxf(hmax, h);
    }
    float fc = 0.0f, fr = 0.0f, gc = 0.0f, gr = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        fc += fabsf(fmaf(-gmin, P.nmp_f[k], P.du_f[k]));
        gc += fabsf(fmaf(-gmax, P.nmp_f[k], P.du_f[k]));
        fr += fabsf(fmaf(-hmin, P.nmp_f[k], P.dv_f[k]));
        gr += fabsf(fmaf(-hmax, P.nmp_f[k], P.dv_f[k]));
    }
    int i0 = 0, i1 = C - 1, j0 = 0, j1 = R - 1;
    if (!bad) pixel_rect(gmin + oc, gmax + oc, hmin + orow, hmax + orow, R, C, i0, i1, j0, j1);
    B.nc[s] = nc;
    B.nr[s] = nr;
    B.dn[s] = dn;
    fc = bad ? 3.0e38f : 0.5f * fmaxf(fc, gc);
    fr = bad ? 3.0e38f : 0.5f * fmaxf(fr, gr);
    // whether every cell's pixels fit a run: those of a larger rectangle by
    // the bound on the shadow where the brick comes nearest to the source
    const float near = dn - 8.0f * P.hn_f;
    const bool runs = (i1 - i0 < RUN_MAX && j1 - j0 < RUN_MAX) ||
                      (near > 0.0f && fmaxf(fc, fr) <= 0.5f * (RUN_MAX - 4) * near);
    B.fc[s] = fc;
    B.fr[s] = fr;
    B.i0[s] = i0;
    B.j0[s] = j0;
    B.w[s] = i1 - i0 + 1;
    B.h[s] = j1 - j0 + 1;
    const int lines = (i1 - i0 + 1) * (j1 - j0 + 1);  // 0 for a view that misses the detector
    B.own[s] = !runs ? half + 2 : lines <= half ? lines : half + 1;
}

// Three (degree 3, at most 168 VGPRs) or four (lower degrees, 128) waves per
// SIMD keep as many blocks on a CU, to hide a batch's set-up between its
// barriers behind other blocks' integration.
template <int n, bool SHARED>
__global__ void __launch_bounds__((CellGather<n, SHARED>::threads))
__attribute__((amdgpu_waves_per_eu((CellGather<n, SHARED>::waves))))
backproject_cells_kernel(const float *__restrict__ y, int N0, int N1, int N2, const float *__restrict__ geom,
                         const ViewProj *__restrict__ vps, int kind, int V, int R, int C, int mz0, int L,
                         typename CellGather<n, SHARED>::Part *__restrict__ T) {
    constexpr int NB = n + 1;
    constexpr int qoff = CellBasis<n>::qoff;
    constexpr double kap = (double)Degree<n>::kap;
    constexpr int THREADS = CellGather<n, SHARED>::threads, SX = CellGather<n, SHARED>::sx, SY = CellGather<n, SHARED>::sy;
    constexpr int BATCH_VIEWS = CellGather<n, SHARED>::batch, RING = 2 * BATCH_VIEWS;  // queued runs per thread
    constexpr int MOMENTS = SHARED ? NB * NB : NB * NB * NB;  // of a thread
    constexpr int HALF = CellGather<n, SHARED>::half;
    // A batch's set-up (records, line table, queueing) is short dependent
    // chains ending in a barrier; the integration is long runs of
    // independent FMAs.  Raising a wave's priority for the set-up lets each
    // block reach its barrier sooner while the other blocks on the CU keep
    // the FMA pipes busy (degrees 1-3; the degree-0 kernel, whose
    // integration is short, runs faster without).
    constexpr int PRIO = CellGather<n, SHARED>::setup_prio;
    const auto prio_setup = [] {
        if constexpr (PRIO > 0) __builtin_amdgcn_s_setprio(PRIO);
    };
    const auto prio_integrate = [] {
        if constexpr (PRIO > 0) __builtin_amdgcn_s_setprio(0);
    };
    static_assert(sizeof(CellRay) == 40, "line record size assumed by the LDS budget");
    __shared__ CellRay rays[2 * HALF];
    __shared__ uint32_t ring[RING * THREADS];  // per-thread queue of runs
    __shared__ BrickViews bv;
    __shared__ int flat_batch[2];  // last batch with a line parallel to an axis, per half
    const int M0 = N0 + n, M1 = N1 + n;  // cells per row / column
    const int nbx = (M0 + GX - 1) / GX, nby = (M1 + GY - 1) / GY, nbz = (L + GZ - 1) / GZ;
    const int nbricks = nbx * nby * nbz;
    const int part = SHARED ? blockIdx.x & 3 : 0;  // quarter of the brick
    const int b = SHARED ? blockIdx.x >> 2 : xcd_remap(blockIdx.x, nbricks);
    const int bx = b % nbx, by = (b / nbx) % nby, bz = b / (nbx * nby);
    const int tid = threadIdx.x, lane = tid & 63;
    const int ox = (part & 1) * SX, oy = (part >> 1) * SY;
    const int cell = SHARED ? lane : tid, q3 = SHARED ? tid >> 6 : 0;  // q3: the wave's power of u3
    const int tx = ox + cell % SX, ty = oy + (cell / SX) % SY, tz = cell / (SX * SY);
    const int c0 = bx * GX + tx, c1 = by * GY + ty, c2 = bz * GZ + tz;  // cell, chunk-relative
    const bool mine = c0 < M0 && c1 < M1 && c2 < L;
    if (SHARED && (bx * GX + ox >= M0 || by * GY + oy >= M1)) return;  // a quarter outside the volume
    // first cell of the brick in index units (cell K spans [K + kap, K + kap + 1]
    // in coordinates x + (N - 1)/2), and the brick centre in world coordinates
    const int mlo = -qoff - n;
    const double centre[3] = {(double)(mlo + bx * GX) + kap - 0.5 * (N0 - 1) + 0.5 * GX,
                              (double)(mlo + by * GY) + kap - 0.5 * (N1 - 1) + 0.5 * GY,
                              (double)(mz0 + bz * GZ) + kap - 0.5 * (N2 - 1) + 0.5 * GZ};
    // this cell's low corner relative to the brick centre (exact)
    const float lo[3] = {(float)tx - 0.5f * GX, (float)ty - 0.5f * GY, (float)tz - 0.5f * GZ};
    const float oc = 0.5f * (float)(C - 1), orow = 0.5f * (float)(R - 1);
    float acc[MOMENTS];
#pragma unroll
    for (int e = 0; e < MOMENTS; ++e) acc[e] = 0.0f;

    // This thread's queue: a ring of runs, oldest first, the next one to
    // start in slot qhead; the run being consumed is in registers (next
    // entry, columns and rows left).  `count` entries are left in all, the
    // oldest `nolder` of them in the half that is not being filled.
    int qhead = 0, qtail = 0, count = 0, nolder = 0;
    int ent = 0, cleft = 0, rleft = 0, cols = 0, jump = 0;
    bool flat = false, flat_other = false;  // such a line in either half, in the half filled last
    // integrate up to `rounds` of this thread's oldest entries
    auto drain = [&](int rounds) {
        const int npop = min(rounds, count);
        for (int k = 0; k < npop; ++k) {
            if (rleft == 0) {  // start the next run
                const uint32_t d = ring[(qhead & (RING - 1)) * THREADS + tid];
                ++qhead;
                ent = (int)(d & 1023u);
                cols = (int)((d >> 10) & 63u) + 1;
                rleft = (int)((d >> 16) & 63u) + 1;
                jump = (int)(d >> 22) + 1 - cols;  // from a row's last entry to the next row's first, less 1
                cleft = cols;
            }
            const int cur = ent;
            --cleft;
            const bool wrap = cleft == 0;
            ent += wrap ? jump + 1 : 1;
            cleft = wrap ? cols : cleft;
            rleft -= wrap ? 1 : 0;
            integrate_hit<n, SHARED>(rays[cur], lo, flat, q3, acc);
        }
        count -= npop;
        nolder = max(nolder - npop, 0);
    };
    auto wave_max = [](int x) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) x = max(x, __shfl_xor(x, m));
        return x;
    };

    // block-uniform: batch number, next view, first column and row of its
    // next segment (a larger view), views whose records are in LDS
    int batch = 0, v = 0, si = 0, sj = 0, rec0 = 0, rec1 = 0;
    if (tid < 2) flat_batch[tid] = -1;
    while (true) {
        prio_setup();
        if (v + BATCH_VIEWS > rec1 && rec1 < V) {
            // records of the next views (every wave is past its reads of the
            // old ones: they precede the last barrier)
            rec0 = v;
            rec1 = min(v + BV_CHUNK, V);
            if (tid < rec1 - rec0) brick_view(vps[rec0 + tid], centre, ox, SX, oy, SY, R, C, HALF, bv, tid);
            __syncthreads();
        }
        // lane l < BATCH_VIEWS holds view v + l: its pixel rectangle, and the
        // lines of the views before it
        const int lv = max(min(v - rec0 + (lane & (BATCH_VIEWS - 1)), rec1 - rec0 - 1), 0);
        int vi0 = bv.i0[lv], vj0 = bv.j0[lv];
        int W = bv.w[lv], H = bv.h[lv];
        const int own = bv.own[lv];
        int upto = own;                           // inclusive sum over lanes 0 .. l
#pragma unroll
        for (int m = 1; m < BATCH_VIEWS; m <<= 1) {
            const int t = __shfl_up(upto, m, BATCH_VIEWS);
            upto += (lane & (BATCH_VIEWS - 1)) >= m ? t : 0;
        }
        const bool fits = lane < BATCH_VIEWS && v + lane < V && upto <= HALF;
        int K = __popcll(__ballot(fits));  // views in this batch (the sums do not decrease)
        // a view too large for a batch comes alone, in segments of whole rows
        // (of columns, for a row wider than that); direct: not queued
        const bool done = v >= V, large = K == 0, direct = __builtin_amdgcn_readlane(own, 0) > HALF + 1;
        // every wave retires its entries of the half that is refilled; before
        // a segment that does not go through the queues and at the end, all
        prio_integrate();
        int rounds = wave_max(nolder);
        if (done || direct) rounds = INT32_MAX;
        drain(rounds);
        if (done) break;
        if (batch >= 2) __syncthreads();
        prio_setup();
        const int half = (batch & 1) * HALF;
        nolder = count;  // every queued entry is now in the older half
        int tb = upto - own, lines;
        const int vb = v;
        if (large) {
            const int BW = __builtin_amdgcn_readlane(W, 0), BH = __builtin_amdgcn_readlane(H, 0);
            const int scols = min(BW, HALF), srows = HALF / scols;
            vi0 += si;
            vj0 += sj;
            W = min(scols, BW - si);
            H = min(srows, BH - sj);
            tb = 0;
            lines = W * H;
            K = 1;
            si += scols;
            if (si >= BW) {
                si = 0;
                sj += srows;
                if (sj >= BH) {
                    sj = 0;
                    ++v;
                }
            }
        } else {
            lines = __builtin_amdgcn_readlane(upto, K - 1);
            v += K;
        }
        for (int base = 0; base < lines; base += THREADS) {
            const int t = base + tid;
            int idx = 0;  // the view of line t
            for (int k = 1; k < K; ++k) idx += t >= __builtin_amdgcn_readlane(tb, k) ? 1 : 0;
            const int w = __shfl(W, idx), ti = __shfl(vi0, idx), tj = __shfl(vj0, idx), tt = t - __shfl(tb, idx);
            if (t < lines) {
                // integer quotient by a float reciprocal: (a + 1/2) / b is at
                // least 1/(2b) away from an integer, far more than its rounding
                const int q = (int)(((float)tt + 0.5f) * __builtin_amdgcn_rcpf((float)w));
                const int jj = tj + q, ii = ti + (tt - q * w), vv = vb + idx;
                if (fill_cellray(rays[half + t], geom + 12 * vv, kind, R, C, jj, ii, centre,
                                 y[((int64_t)vv * R + jj) * C + ii]))
                    flat_batch[batch & 1] = batch;
            }
        }
        for (int k = 0; k < K; ++k) {
            const int w = __builtin_amdgcn_readlane(W, k), h = __builtin_amdgcn_readlane(H, k);
            if (w <= 0 || h <= 0) continue;
            const ViewProj &P = vps[vb + k];
            const int s = vb + k - rec0;
            const float d0 = lo[0] + 0.5f, d1 = lo[1] + 0.5f, d2 = lo[2] + 0.5f;
            const float nu = fmaf(d2, P.du_f[2], fmaf(d1, P.du_f[1], fmaf(d0, P.du_f[0], bv.nc[s])));
            const float nv = fmaf(d2, P.dv_f[2], fmaf(d1, P.dv_f[1], fmaf(d0, P.dv_f[0], bv.nr[s])));
            const float den = fmaf(d2, P.nmp_f[2], fmaf(d1, P.nmp_f[1], fmaf(d0, P.nmp_f[0], bv.dn[s])));
            const float lam = __builtin_amdgcn_rcpf(den), rr = __builtin_amdgcn_rcpf(den - P.hn_f);
            const bool open = !(den > P.hn_f);  // a corner on or behind the source plane: no bounded shadow
            // relative to the rectangle's first pixel
            const float cc = fmaf(lam, nu, P.gac_f + (oc - (float)__builtin_amdgcn_readlane(vi0, k)));
            const float cr = fmaf(lam, nv, P.gar_f + (orow - (float)__builtin_amdgcn_readlane(vj0, k)));
            const float ec = fmaf(bv.fc[s], rr, PIX_MARGIN), er = fmaf(bv.fr[s], rr, PIX_MARGIN);
            const float wf = (float)(w - 1), hf = (float)(h - 1);
            const float fi0 = open ? 0.0f : fmaxf(ceilf(cc - ec), 0.0f), fi1 = open ? wf : fminf(floorf(cc + ec), wf);
            const float fj0 = open ? 0.0f : fmaxf(ceilf(cr - er), 0.0f), fj1 = open ? hf : fminf(floorf(cr + er), hf);
            if (mine && fi0 <= fi1 && fj0 <= fj1) {
                const int ni = (int)(fi1 - fi0), nj = (int)(fj1 - fj0);  // columns and rows, less 1
                const int first = half + __builtin_amdgcn_readlane(tb, k) + (int)fmaf(fj0, (float)w, fi0);
                if (direct) {  // the queue is empty: straight to the registers
                    ent = first;
                    cols = cleft = ni + 1;
                    rleft = nj + 1;
                    jump = w - cols;
                } else {
                    ring[(qtail & (RING - 1)) * THREADS + tid] =
                        (uint32_t)first | (uint32_t)ni << 10 | (uint32_t)nj << 16 | (uint32_t)(w - 1) << 22;
                    ++qtail;
                }
                count += (ni + 1) * (nj + 1);
            }
        }
        __syncthreads();  // the half is filled; every record of this batch has been read
        const bool now = flat_batch[batch & 1] == batch;
        flat = now || flat_other;
        flat_other = now;
        ++batch;
    }
    // moments -> per-basis integrals: apply the blending map along each axis
    if constexpr (n > 0) {
#pragma unroll
        for (int i = 0; i < MOMENTS / NB; ++i) {  // axis 1: index (i, p1)
            float t[NB];
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                t[a] = 0.0f;
#pragma unroll
                for (int p = 0; p < NB; ++p) t[a] = fmaf(blend_u<n>(a, p), acc[i * NB + p], t[a]);
            }
#pragma unroll
            for (int a = 0; a < NB; ++a) acc[i * NB + a] = t[a];
        }
#pragma unroll
        for (int i3 = 0; i3 < MOMENTS / (NB * NB); ++i3)  // axis 2: index (i3, p2, a1)
#pragma unroll
            for (int i1 = 0; i1 < NB; ++i1) {
                float t[NB];
#pragma unroll
                for (int a = 0; a < NB; ++a) {
                    t[a] = 0.0f;
#pragma unroll
                    for (int p = 0; p < NB; ++p) t[a] = fmaf(blend_u<n>(a, p), acc[(i3 * NB + p) * NB + i1], t[a]);
                }
#pragma unroll
                for (int a = 0; a < NB; ++a) acc[(i3 * NB + a) * NB + i1] = t[a];
            }
        if constexpr (SHARED) {  // axis 3: the waves' moments through the line table's memory
            static_assert(sizeof rays >= NB * NB * NB * 64 * 4, "room for a block's moments");
            float *x = reinterpret_cast<float *>(rays);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB * NB; ++i) x[(q3 * NB * NB + i) * 64 + lane] = acc[i];
            __syncthreads();
            float w[NB];
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                w[p] = blend_u<n>(0, p);
#pragma unroll
                for (int a = 1; a < NB; ++a) w[p] = q3 == a ? blend_u<n>(a, p) : w[p];
            }
#pragma unroll
            for (int i = 0; i < NB * NB; ++i) {
                acc[i] = 0.0f;
#pragma unroll
                for (int p = 0; p < NB; ++p) acc[i] = fmaf(w[p], x[(p * NB * NB + i) * 64 + lane], acc[i]);
            }
        } else
#pragma unroll
        for (int i = 0; i < NB * NB; ++i) {  // axis 3: index (p3, i)
            float t[NB];
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                t[a] = 0.0f;
#pragma unroll
                for (int p = 0; p < NB; ++p) t[a] = fmaf(blend_u<n>(a, p), acc[p * NB * NB + i], t[a]);
            }
#pragma unroll
            for (int a = 0; a < NB; ++a) acc[a * NB * NB + i] = t[a];
        }
    }
    // this block's part of each coefficient: its cells' entries summed in
    // FP64, entry by entry, (n+1)^2 entries of every cell at a time through
    // the line table's memory (all of them when the waves share the moments)
    constexpr int NC = CellGather<n, SHARED>::coeffs, CELLS = SHARED ? 64 : 256;
    constexpr int PER = (NC + THREADS - 1) / THREADS, EX = SX + n, EY = SY + n;
    static_assert(sizeof rays >= (SHARED ? NB : 1) * NB * NB * CELLS * 4, "room for the entries");
    float *x = reinterpret_cast<float *>(rays);
    double sum[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) sum[r] = 0.0;
#pragma unroll
    for (int a3 = 0; a3 < NB; ++a3) {
        if (!SHARED || a3 == 0) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB * NB; ++i)
                x[((SHARED ? q3 * NB * NB : 0) + i) * CELLS + cell] = acc[SHARED ? i : a3 * NB * NB + i];
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int e = tid + r * THREADS, i = e % EX, j = (e / EX) % EY, z = e / (EX * EY) - a3;
            if (e >= NC || z < 0 || z >= GZ) continue;
            // all loads at once; a cell outside the block adds 0 (branches
            // around each load cost a call of one view over 33 x 31 x 40
            // 24.5 instead of 21.9 us at degree 3, 16.5 and 14.8 at degree 2)
            const float *at = x + (SHARED ? a3 * NB * NB : 0) * CELLS;
            float t[NB][NB];
#pragma unroll
            for (int a2 = 0; a2 < NB; ++a2)
#pragma unroll
                for (int a1 = 0; a1 < NB; ++a1) {
                    const bool in = (unsigned)(j - a2) < (unsigned)SY && (unsigned)(i - a1) < (unsigned)SX;
                    const float v = at[in ? (a2 * NB + a1) * CELLS + (z * SY + j - a2) * SX + i - a1 : 0];
                    t[a2][a1] = in ? v : 0.0f;
                }
#pragma unroll
            for (int a2 = 0; a2 < NB; ++a2)
#pragma unroll
                for (int a1 = 0; a1 < NB; ++a1) sum[r] += (double)t[a2][a1];
        }
    }
    const int qx = SHARED ? 2 * bx + (part & 1) : bx, qy = SHARED ? 2 * by + (part >> 1) : by;
    const int nqx = SHARED ? 2 * nbx : nbx, nqy = SHARED ? 2 * nby : nby;
    auto *out = T + (((int64_t)bz * nqy + qy) * nqx + qx) * CellGather<n, SHARED>::record;
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (tid + r * THREADS < NC) out[tid + r * THREADS] = (typename CellGather<n, SHARED>::Part)sum[r];
}

// Pass 2: coefficient k (layer k2 in [qz0, qz1]) adds its parts of the blocks
// that hold cells of its support (up to two per axis), in FP64.
template <int n, bool SHARED>
__global__ void __launch_bounds__(256) cells_to_coeffs_kernel(const typename CellGather<n, SHARED>::Part *__restrict__ T,
                                                              int N0, int N1, int mz0, int qz0, int qz1,
                                                              float *__restrict__ c) {
    constexpr int qoff = CellBasis<n>::qoff;
    using G = CellGather<n, SHARED>;
    const int64_t per = (int64_t)N0 * N1;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= per * (qz1 - qz0 + 1)) return;
    const int k2 = qz0 + (int)(idx / per);
    const int rem = (int)(idx % per);
    const int k1 = rem / N0, k0 = rem % N0;
    const int nqx = (N0 + n + GX - 1) / GX * (GX / G::sx), nqy = (N1 + n + GY - 1) / GY * (GY / G::sy);
    // cells of the support, relative to the volume's (the chunk's) first:
    // k0 .. k0 + n, k1 .. k1 + n, z .. z + n
    const int z = k2 - qoff - mz0 - n;
    // one or two blocks per axis: all loads at once, a block that is not there
    // adds 0 (one after the other, each waited for: one view over 33 x 31 x 40
    // 21.9 instead of 20.1 us at degree 3, 14.8 and 13.4 at degree 2)
    static_assert(n < G::sx && n < G::sy && n < GZ + 1, "at most two blocks per axis");
    const int bx0 = k0 / G::sx, by0 = k1 / G::sy, bz0 = z / GZ;
    const bool mx = (k0 + n) / G::sx != bx0, my = (k1 + n) / G::sy != by0, mz = (z + n) / GZ != bz0;
    typename G::Part t[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int qx = q & 1, qy = (q >> 1) & 1, qz = q >> 2;
        const bool in = (!qx || mx) && (!qy || my) && (!qz || mz);
        const int bx = bx0 + (in ? qx : 0), by = by0 + (in ? qy : 0), bz = bz0 + (in ? qz : 0);
        const auto v = T[(((int64_t)bz * nqy + by) * nqx + bx) * G::record +
                         ((z + n - bz * GZ) * (G::sy + n) + k1 + n - by * G::sy) * (G::sx + n) + k0 + n - bx * G::sx];
        t[q] = in ? v : 0;
    }
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s += t[q];
    c[(int64_t)k2 * per + rem] = (float)s;
}

// ---------------------------------------------------------------------------
// Footprint of arbitrary pairs (diagnostics): w unit, x any point of the
// line relative to the basis centre.
// ---------------------------------------------------------------------------
template <int n>
__global__ void footprint_kernel(const float *__restrict__ dirs, const float *__restrict__ offs, int count,
                                 float *__restrict__ out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    double w[3], x[3];
    for (int a = 0; a < 3; ++a) { w[a] = dirs[3 * k + a]; x[a] = offs[3 * k + a]; }
    int d, i1, i2;
    dominant_axis(w, d, i1, i2);
    const double wd = pick3(w, d);
    if (wd == 0.0) { out[k] = 0.0f; return; }
    const double r1 = pick3(w, i1) / wd, r2 = pick3(w, i2) / wd;
    const Slopes S = make_slopes((float)r1, (float)r2);
    const double xd = pick3(x, d);
    const float u1 = (float)(pick3(x, i1) - xd * r1), u2 = (float)(pick3(x, i2) - xd * r2);
    const double nrm = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
    out[k] = footprint_slab<n>(S, u1, u2) * (float)(nrm / fabs(wd));
}

// ---------------------------------------------------------------------------
// FP64-accumulated inner product (two passes, fixed grid: deterministic),
// FP64 ratio, FP32 vector updates with a device scalar.
// ---------------------------------------------------------------------------
constexpr int DOT_BLOCKS = 1024, DOT_THREADS = 256;

__global__ void __launch_bounds__(DOT_THREADS) dot_partial_kernel(const float *__restrict__ a,
                                                                  const float *__restrict__ b, int64_t n,
                                                                  double *__restrict__ part) {
    __shared__ double red[DOT_THREADS];
    double s = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        s = fma((double)a[i], (double)b[i], s);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = DOT_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(DOT_THREADS) dot_final_kernel(const double *__restrict__ part, int np,
                                                                double *__restrict__ out) {
    __shared__ double red[DOT_THREADS];
    double s = 0.0;
    for (int i = threadIdx.x; i < np; i += DOT_THREADS) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = DOT_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

__global__ void ratio_kernel(const double *__restrict__ num, const double *__restrict__ den,
                             double *__restrict__ out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const double dd = *den;
        *out = dd != 0.0 ? *num / dd : 0.0;
    }
}

__global__ void axpy_kernel(const double *__restrict__ alpha, float sign, const float *__restrict__ x,
                            float *__restrict__ yv, int64_t n) {
    const float a = sign * (float)(*alpha);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        yv[i] = fmaf(a, x[i], yv[i]);
}

__global__ void xpay_kernel(const double *__restrict__ beta, const float *__restrict__ x, float *__restrict__ yv,
                            int64_t n) {
    const float bt = (float)(*beta);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        yv[i] = fmaf(bt, yv[i], x[i]);
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
template <int n, int LPL, bool WIDE>
static void launch_walk(const LaunchArgs &a, const float *cz, const float *cx, int which, hipStream_t st) {
    const int tR = (a.R + 15) / 16, tC = (a.C + 15) / 16;
    const auto launch = [&](int v0, int V) {
        const int64_t nb = LPL == 1 ? fwd_blocks(tR, tC, V) : (int64_t)tR * tC * V * LPL;
        hipLaunchKernelGGL((project_kernel<n, LPL, WIDE>), dim3((unsigned)nb), dim3(256), 0, st, cz, cx, a.N[0],
                           a.N[1], a.N[2], a.geom + 12 * (int64_t)v0, a.kind, V, a.R, a.C,
                           a.sino + (int64_t)v0 * a.R * a.C, which, fwd_views(V));
    };
    if (LPL == 1) fwd_in_pieces(tR, tC, a.V, launch);
    else launch(0, a.V);
}

template <int n>
static hipError_t launch_project_n(const LaunchArgs &a, hipStream_t st) {
    constexpr int P = FWD_PAD(n);
    const int64_t Sx = a.N[0] + 2 * P, Sy = a.N[1] + 2 * P, Sz = a.N[2] + 2 * P, padded = Sx * Sy * Sz;
    if (!a.scratch || a.scratch_floats < padded) return hipErrorInvalidValue;
    const int64_t zb = ((Sx + PAD_T - 1) / PAD_T) * ((Sz + PAD_T - 1) / PAD_T) * Sy;
    if (zb > INT32_MAX || !fwd_launch_views((a.R + 15) / 16, (a.C + 15) / 16, a.V)) return hipErrorInvalidValue;
    const int64_t tiles = (int64_t)((a.R + 15) / 16) * ((a.C + 15) / 16) * a.V;
    const int64_t shared = a.spacing > FWD_SPARSE ? FWD_SPARSE_TILES[n] : FWD_SHARED_TILES[n][padded > FWD_SHARED_FLOATS];
    const auto walk = [&](const float *cz, const float *cx, int which) {
        if (padded > (int64_t)1 << 30) launch_walk<n, 1, true>(a, cz, cx, which, st);
        else if (tiles <= shared) launch_walk<n, 4, false>(a, cz, cx, which, st);
        else launch_walk<n, 1, false>(a, cz, cx, which, st);
    };
    // the x-fastest copy, for the views that walk it, beside the z-fastest
    // one or, where the scratch holds one, in its place after a launch for
    // the views of the other (stream order)
    const bool both = a.scratch_floats >= 2 * padded;
    float *cz = a.scratch, *cx = !a.walks_x ? nullptr : both ? a.scratch + padded : a.scratch;
    hipLaunchKernelGGL(pad_volume_zfast_kernel, dim3((unsigned)zb), dim3(256), 0, st, a.coeffs, a.N[0], a.N[1], a.N[2],
                       P, cz);
    if (!cx) {
        walk(cz, cx, 2);
        return hipGetLastError();
    }
    if (!both) walk(cz, cx, 0);
    hipLaunchKernelGGL(pad_volume_kernel, dim3((unsigned)std::min<int64_t>((padded + 255) / 256, 65536)), dim3(256), 0,
                       st, a.coeffs, a.N[0], a.N[1], a.N[2], P, cx);
    walk(cz, cx, both ? 2 : 1);
    return hipGetLastError();
}

int64_t project_quad_scratch_floats(int degree, const int N[3]) {
    const int64_t P = degree + 1;
    return (N[0] + 2 * P) * (N[1] + 2 * P) * (N[2] + 2 * P);
}

float project_quad_spacing(const float *vec, int kind) {
    const float *s = vec, *d0 = vec + 3, *u = vec + 6, *v = vec + 9;
    const double cx = (double)u[1] * v[2] - (double)u[2] * v[1], cy = (double)u[2] * v[0] - (double)u[0] * v[2],
                 cz = (double)u[0] * v[1] - (double)u[1] * v[0];
    const auto norm = [](double x, double y, double z) { return sqrt(x * x + y * y + z * z); };
    const double pitch = sqrt(norm(cx, cy, cz));
    if (kind == 0) return (float)pitch;
    const double sd = norm((double)d0[0] - s[0], (double)d0[1] - s[1], (double)d0[2] - s[2]);
    return (float)(pitch * norm(s[0], s[1], s[2]) / sd);
}

int project_quad_copies(int degree, const int N[3], bool walks_x) {
    return walks_x && project_quad_scratch_floats(degree, N) <= FWD_BOTH_FLOATS ? 2 : 1;
}

template <int n> static bool walks_x_n(const float *vecs, int V, int kind) {
    for (int v = 0; v < V; ++v)
        if (view_walk<n>(vecs + 12 * (int64_t)v, kind).xcopy) return true;
    return false;
}

bool project_quad_walks_x(int degree, const float *vecs, int V, int kind) {
    // the contraction order, which keeps a view from the x-fastest copy, is
    // the same at every degree but 0
    return degree == 0 ? walks_x_n<0>(vecs, V, kind) : walks_x_n<1>(vecs, V, kind);
}

// Whether the adjoint of a volume shares each cell's moments, and the floats
// of the table per GZ cell layers.
template <int n> static bool cells_shared(const int N[3]) {
    const int64_t nb = (int64_t)((N[0] + n + GX - 1) / GX) * ((N[1] + n + GY - 1) / GY) * ((N[2] + n + GZ - 1) / GZ);
    return n >= 2 && nb <= SHARED_BRICKS;
}
template <int n> static int64_t cell_table_floats(const int N[3]) {
    const int64_t bricks = (int64_t)((N[0] + n + GX - 1) / GX) * ((N[1] + n + GY - 1) / GY);
    const int64_t record = cells_shared<n>(N) ? 4 * CellGather<n, true>::record : CellGather<n, false>::record;
    return bricks * record * (int64_t)(sizeof(typename CellGather<n, false>::Part) / sizeof(float));
}

template <int n> static int64_t scratch_floats_n(const int N[3], int64_t limit) {
    const int64_t slab = cell_table_floats<n>(N);
    // at least 4 (n + 1) layers per chunk, so that chunking re-does at most
    // a quarter of the cell layers
    const int64_t floor_layers = std::min<int64_t>(N[2] + n, 4 * (n + 1));
    return std::min(slab * ((N[2] + n + GZ - 1) / GZ), std::max(limit, slab * ((floor_layers + GZ - 1) / GZ)));
}

int64_t backproject_quad_scratch_floats(int degree, const int N[3], int64_t limit) {
    switch (degree) {
    case 0: return scratch_floats_n<0>(N, limit);
    case 1: return scratch_floats_n<1>(N, limit);
    case 2: return scratch_floats_n<2>(N, limit);
    default: return scratch_floats_n<3>(N, limit);
    }
}

template <int n, bool SHARED>
static hipError_t launch_backproject_cells(const LaunchArgs &a, hipStream_t st) {
    constexpr int qoff = CellBasis<n>::qoff;
    const int M0 = a.N[0] + n, M1 = a.N[1] + n, M2 = a.N[2] + n;
    const int Lmax = (int)std::min<int64_t>(M2, a.scratch_floats / cell_table_floats<n>(a.N) * GZ);
    if (!a.scratch || Lmax <= n) return hipErrorInvalidValue;
    auto *T = reinterpret_cast<typename CellGather<n, SHARED>::Part *>(a.scratch);
    const int mlo = -qoff - n;
    const int64_t plane = (int64_t)a.N[0] * a.N[1];
    for (int s = mlo;;) {
        const int L = std::min(Lmax, mlo + M2 - s);
        const int nb = ((M0 + GX - 1) / GX) * ((M1 + GY - 1) / GY) * ((L + GZ - 1) / GZ);
        hipLaunchKernelGGL((backproject_cells_kernel<n, SHARED>), dim3(SHARED ? 4 * nb : nb),
                           dim3(CellGather<n, SHARED>::threads), 0, st, a.sino_in, a.N[0], a.N[1], a.N[2], a.geom,
                           a.vproj, a.kind, a.V, a.R, a.C, s, L, T);
        const int qz0 = s + qoff + n, qz1 = std::min(s + L - 1 + qoff, a.N[2] - 1);
        if (qz1 >= qz0) {
            const int64_t cnt = plane * (qz1 - qz0 + 1);
            hipLaunchKernelGGL((cells_to_coeffs_kernel<n, SHARED>), dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0,
                               st, T, a.N[0], a.N[1], s, qz0, qz1, a.coeffs_out);
        }
        if (s + L >= mlo + M2) break;
        s += L - n;
    }
    return hipGetLastError();
}

template <int n>
static hipError_t launch_backproject_n(const LaunchArgs &a, hipStream_t st) {
    if constexpr (n >= 2)
        if (cells_shared<n>(a.N)) return launch_backproject_cells<n, true>(a, st);
    return launch_backproject_cells<n, false>(a, st);
}

hipError_t launch_project_quad(int degree, const LaunchArgs &a, hipStream_t st) {
    switch (degree) {
    case 0: return launch_project_n<0>(a, st);
    case 1: return launch_project_n<1>(a, st);
    case 2: return launch_project_n<2>(a, st);
    case 3: return launch_project_n<3>(a, st);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Allocation-free forward: a file-scope device array holds the view vectors
// and the zero-padded coefficients.  Host code never passes `scratch` itself
// to a kernel (in host code the name is a host-side stand-in); it asks the
// runtime, once per device with that device current, for the array's device
// address and passes that.
// ---------------------------------------------------------------------------
static __device__ __align__(256) float scratch[STATIC_SCRATCH_FLOATS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t static_scratch_address(int device, float **ptr) {
    *ptr = nullptr;
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = static_cast<float *>(p);
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_backproject_quad(int degree, const LaunchArgs &a, hipStream_t st) {
    switch (degree) {
    case 0: return launch_backproject_n<0>(a, st);
    case 1: return launch_backproject_n<1>(a, st);
    case 2: return launch_backproject_n<2>(a, st);
    case 3: return launch_backproject_n<3>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_footprint_quad(int degree, const float *dirs, const float *offs, int count, float *out,
                                 hipStream_t st) {
    const int nb = (count + 255) / 256;
    if (count == 0) return hipSuccess;
    switch (degree) {
    case 0: hipLaunchKernelGGL(footprint_kernel<0>, dim3(nb), dim3(256), 0, st, dirs, offs, count, out); break;
    case 1: hipLaunchKernelGGL(footprint_kernel<1>, dim3(nb), dim3(256), 0, st, dirs, offs, count, out); break;
    case 2: hipLaunchKernelGGL(footprint_kernel<2>, dim3(nb), dim3(256), 0, st, dirs, offs, count, out); break;
    case 3: hipLaunchKernelGGL(footprint_kernel<3>, dim3(nb), dim3(256), 0, st, dirs, offs, count, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_dot(const float *a, const float *b, int64_t n, double *partials, double *out, hipStream_t st) {
    hipLaunchKernelGGL(dot_partial_kernel, dim3(DOT_BLOCKS), dim3(DOT_THREADS), 0, st, a, b, n, partials);
    hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(DOT_THREADS), 0, st, partials, DOT_BLOCKS, out);
    return hipGetLastError();
}

int dot_partials_needed() { return DOT_BLOCKS; }

hipError_t launch_ratio(const double *num, const double *den, double *out, hipStream_t st) {
    hipLaunchKernelGGL(ratio_kernel, dim3(1), dim3(64), 0, st, num, den, out);
    return hipGetLastError();
}

static int vec_blocks(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (int)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

hipError_t launch_axpy(const double *alpha, float sign, const float *x, float *yv, int64_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(axpy_kernel, dim3(vec_blocks(n)), dim3(256), 0, st, alpha, sign, x, yv, n);
    return hipGetLastError();
}

hipError_t launch_xpay(const double *beta, const float *x, float *yv, int64_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(xpay_kernel, dim3(vec_blocks(n)), dim3(256), 0, st, beta, x, yv, n);
    return hipGetLastError();
}

}  // namespace ss
