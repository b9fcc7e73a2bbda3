// ss_traverse.hpp -- launch-order and detector-mapping helpers shared by the
// quadrature and network kernels.
#pragma once

#include "ss_launch.hpp"
#include "ss_math.hpp"

namespace ss {

// ---------------------------------------------------------------------------
// XCD-aware block order: consecutive hardware block ids go round-robin over
// the 8 XCDs, each with its own L2.  Every XCD gets runs of XCD_RUN
// neighbouring tiles (which read overlapping data through its L2), the runs
// dealt eight at a time, each eight rotated against the last ones, so that
// every XCD works all over the volume and they end together.  With a contiguous eighth of the
// volume for each XCD the chip was idle for 5 to 14 % of an adjoint: cone_256
// degree 3 159 -> 151 ms, 2 82.5 -> 77.9, 1 56.0 -> 52.5, 0 46.2 -> 42.6; 97 x
// 75 x 61 degree 1 0.558 -> 0.514.  Runs of 1, 8, 32: 43.1, 42.6, 42.4 and
// 0.511, 0.515, 0.524 ms.
// A permutation of 0 .. nblocks - 1.
// ---------------------------------------------------------------------------
constexpr int XCD_RUN = 8;
constexpr int xcd_remap(int b, int nblocks) {
    if (b >= nblocks / (8 * XCD_RUN) * (8 * XCD_RUN)) return b;
    const int l = b / 8, e = l / XCD_RUN;
    return (e * 8 + ((b + xcd_rotation(e)) & 7)) * XCD_RUN + l % XCD_RUN;
}

// View and tile of this block; false for a padding slot (a whole block).
__device__ __forceinline__ bool fwd_block_tile(int V, int nv, int tR, int tC, int &v, int &tr, int &tc) {
    return fwd_slot(blockIdx.x, V, nv, tR, tC, v, tr, tc);
}

struct ViewProj {    // detector coordinates of a world point (FP64 set-up)
    double d0[3], s[3], du_s[3], dv_s[3], nrm[3];
    double plane;    // (d0 - s) . nrm  (cone)
    // for make_localproj: o . du_s, o . dv_s, o . nrm with o = s (cone) or d0
    // (parallel), and the FP32 values that do not depend on the centre
    double odu, odv, onm;
    float du_f[3], dv_f[3], nm_f[3];
    float ac_f, ar_f, plane_f;  // (s - d0) . du_s, (s - d0) . dv_s, plane
    int kind;
    // for the knot-cell gather, where both kinds read col = ac + nu / den,
    // row = ar + nv / den: nrm / plane (0 for parallel beams, whose den is 1),
    // half the sum of its magnitudes, and the two additive terms (0 for
    // parallel beams)
    float nmp_f[3], hn_f, gac_f, gar_f;
};

// Continuous pixel coordinates (column, row) of world point X.
// parallel: X = d0 + alpha du + beta dv + t w ;  cone: the detector point
// of the line through the source and X.  Returns false when undefined.
__device__ __forceinline__ bool to_detector(const ViewProj &P, const double X[3], double &col, double &row) {
    double q[3];
    if (P.kind == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = X[k] - P.d0[k];
    } else {
        double dx[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) dx[k] = X[k] - P.s[k];
        const double den = dx[0] * P.nrm[0] + dx[1] * P.nrm[1] + dx[2] * P.nrm[2];
        if (!(den * P.plane > 0.0)) return false;  // X on or behind the source plane
        const double lam = P.plane / den;
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = P.s[k] + lam * dx[k] - P.d0[k];
    }
    col = q[0] * P.du_s[0] + q[1] * P.du_s[1] + q[2] * P.du_s[2];
    row = q[0] * P.dv_s[0] + q[1] * P.dv_s[1] + q[2] * P.dv_s[2];
    return true;
}

// Dual basis: du_s . du = 1, du_s . dv = 0, du_s . m = 0 (m = w or the
// detector normal), likewise dv_s.
__host__ __device__ inline void make_viewproj(const float *__restrict__ e, int kind, ViewProj &P) {
    double du[3], dv[3], m[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        P.s[k] = e[k];
        P.d0[k] = e[3 + k];
        du[k] = e[6 + k];
        dv[k] = e[9 + k];
    }
    P.kind = kind;
    P.nrm[0] = du[1] * dv[2] - du[2] * dv[1];
    P.nrm[1] = du[2] * dv[0] - du[0] * dv[2];
    P.nrm[2] = du[0] * dv[1] - du[1] * dv[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = kind == 0 ? P.s[k] : P.nrm[k];
    P.plane = (P.d0[0] - P.s[0]) * P.nrm[0] + (P.d0[1] - P.s[1]) * P.nrm[1] + (P.d0[2] - P.s[2]) * P.nrm[2];
    // rows of inverse([du dv m]) via cross products
    double c0[3] = {dv[1] * m[2] - dv[2] * m[1], dv[2] * m[0] - dv[0] * m[2], dv[0] * m[1] - dv[1] * m[0]};
    double c1[3] = {m[1] * du[2] - m[2] * du[1], m[2] * du[0] - m[0] * du[2], m[0] * du[1] - m[1] * du[0]};
    const double det = du[0] * c0[0] + du[1] * c0[1] + du[2] * c0[2];
    const double id = det != 0.0 ? 1.0 / det : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        P.du_s[k] = c0[k] * id;
        P.dv_s[k] = c1[k] * id;
    }
    double o[3], sd[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        o[k] = kind == 0 ? P.d0[k] : P.s[k];
        sd[k] = P.s[k] - P.d0[k];
        P.du_f[k] = (float)P.du_s[k];
        P.dv_f[k] = (float)P.dv_s[k];
        P.nm_f[k] = (float)P.nrm[k];
    }
    P.odu = o[0] * P.du_s[0] + o[1] * P.du_s[1] + o[2] * P.du_s[2];
    P.odv = o[0] * P.dv_s[0] + o[1] * P.dv_s[1] + o[2] * P.dv_s[2];
    P.onm = o[0] * P.nrm[0] + o[1] * P.nrm[1] + o[2] * P.nrm[2];
    P.ac_f = (float)(sd[0] * P.du_s[0] + sd[1] * P.du_s[1] + sd[2] * P.du_s[2]);
    P.ar_f = (float)(sd[0] * P.dv_s[0] + sd[1] * P.dv_s[1] + sd[2] * P.dv_s[2]);
    P.plane_f = (float)P.plane;
    const double ip = kind == 0 || P.plane == 0.0 ? 0.0 : 1.0 / P.plane;
    double hn = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        P.nmp_f[k] = (float)(P.nrm[k] * ip);
        hn += 0.5 * (P.nrm[k] * ip < 0.0 ? -P.nrm[k] * ip : P.nrm[k] * ip);
    }
    P.hn_f = (float)hn;
    P.gac_f = kind == 0 ? 0.0f : P.ac_f;
    P.gar_f = kind == 0 ? 0.0f : P.ar_f;
}

// Detector coordinates of points X = c + delta near a centre c, evaluated in
// FP32 for small delta; every term that involves c or the source is formed
// in FP64 once.  With D = c - s (cone) or c - d0 (parallel):
//   parallel: col = D . du_s + delta . du_s
//   cone:     col = (s - d0) . du_s + plane (D . du_s + delta . du_s) / (D . nrm + delta . nrm)
// and likewise for rows with dv_s.
struct LocalProj {
    float du[3], dv[3], nm[3];
    float nc, nr, dn;   // D . du_s, D . dv_s, D . nrm
    float ac, ar;       // (s - d0) . du_s, (s - d0) . dv_s  (cone)
    float plane;
    int kind;
};

// D . du_s = c . du_s - o . du_s in FP64 (three FMA and a difference per
// term); everything else comes from the view's set-up.
__device__ __forceinline__ void make_localproj(const ViewProj &P, const double c[3], LocalProj &L) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        L.du[k] = P.du_f[k];
        L.dv[k] = P.dv_f[k];
        L.nm[k] = P.nm_f[k];
    }
    L.nc = (float)(fma(c[2], P.du_s[2], fma(c[1], P.du_s[1], c[0] * P.du_s[0])) - P.odu);
    L.nr = (float)(fma(c[2], P.dv_s[2], fma(c[1], P.dv_s[1], c[0] * P.dv_s[0])) - P.odv);
    L.dn = (float)(fma(c[2], P.nrm[2], fma(c[1], P.nrm[1], c[0] * P.nrm[0])) - P.onm);
    L.ac = P.ac_f;
    L.ar = P.ar_f;
    L.plane = P.plane_f;
    L.kind = P.kind;
}

// false when X is on or behind the source plane (cone)
__device__ __forceinline__ bool local_to_detector(const LocalProj &L, const float d[3], float &col, float &row) {
    const float nu = fmaf(d[2], L.du[2], fmaf(d[1], L.du[1], fmaf(d[0], L.du[0], L.nc)));
    const float nv = fmaf(d[2], L.dv[2], fmaf(d[1], L.dv[1], fmaf(d[0], L.dv[0], L.nr)));
    if (L.kind == 0) {
        col = nu;
        row = nv;
        return true;
    }
    const float den = fmaf(d[2], L.nm[2], fmaf(d[1], L.nm[1], fmaf(d[0], L.nm[0], L.dn)));
    if (!(den * L.plane > 0.0f)) return false;
    const float lam = L.plane * __builtin_amdgcn_rcpf(den);
    col = fmaf(lam, nu, L.ac);
    row = fmaf(lam, nv, L.ar);
    return true;
}

// Pixel rectangle [i0, i1] x [j0, j1] covering every line that meets the
// box [lo, hi] (whole detector if the projection is undefined).
__device__ __forceinline__ void box_to_pixels(const ViewProj &P, const double lo[3], const double hi[3], int R,
                                              int C, int &i0, int &i1, int &j0, int &j1) {
    double cmin = 1e300, cmax = -1e300, rmin = 1e300, rmax = -1e300;
    bool ok = true;
#pragma unroll
    for (int corner = 0; corner < 8; ++corner) {
        double X[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) X[k] = ((corner >> k) & 1) ? hi[k] : lo[k];
        double cc, rr;
        if (!to_detector(P, X, cc, rr)) ok = false;
        cmin = fmin(cmin, cc); cmax = fmax(cmax, cc);
        rmin = fmin(rmin, rr); rmax = fmax(rmax, rr);
    }
    if (!ok) { i0 = 0; i1 = C - 1; j0 = 0; j1 = R - 1; return; }
    const double oc = 0.5 * (C - 1), orow = 0.5 * (R - 1);
    const double fi0 = floor(cmin + oc) - 1.0, fi1 = ceil(cmax + oc) + 1.0;
    const double fj0 = floor(rmin + orow) - 1.0, fj1 = ceil(rmax + orow) + 1.0;
    if (!(fi1 >= 0.0 && fj1 >= 0.0 && fi0 <= (double)(C - 1) && fj0 <= (double)(R - 1))) {
        i0 = 0; i1 = -1; j0 = 0; j1 = -1;  // empty (also catches NaN)
        return;
    }
    // clamped in FP64 before converting
    i0 = (int)fmax(fi0, 0.0); i1 = (int)fmin(fi1, (double)(C - 1));
    j0 = (int)fmax(fj0, 0.0); j1 = (int)fmin(fj1, (double)(R - 1));
}

}  // namespace ss
