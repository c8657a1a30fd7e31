// Footprint projector pairs -- separable footprint (SF) and distance-driven
// (DD) -- and their rigid-motion gradients (the discrete projectors
// l = A mu, mu = A^T l of Sec. II-C with footprint weights a_ij; gradients by
// Eqs. dis_forward / dis_back: the same weights applied to G_f per voxel and
// to G_b per pixel).
//
// DD replaces the transaxial trapezoid by a unit-height rectangle between
// the projections of the voxel's two boundaries across the view's dominant
// transaxial axis (x if the source's object-frame offset from the volume
// centre has |x| >= |y|, else y), taken at the voxel centre, and the chord
// by the path length h_dom |d| / |d_dom| through the slab along that axis.
// Everything else below is shared.
//
// Footprint of voxel j in one view, with the voxel moved by the pose (the
// view's projective map on voxel indices; FP64 anchors per voxel column and
// view, exact FP32 offsets per voxel, see SfColumn):
//   transaxial: the corners (i +- 1/2, j +- 1/2) of the mid-height
//     cross-section project to columns tau0 <= tau1 <= tau2 <= tau3, the
//     breakpoints of a unit-height trapezoid T(a);
//   axial: the top and bottom centres (k +- 1/2) project to rows
//     [b_lo, b_hi], a unit-height rectangle;
//   amplitude: the chord L_j of the voxel along the line from the source
//     through its centre;
//   a_ij = L_j * int_{a_i - 1/2}^{a_i + 1/2} T * |[b_lo, b_hi] cap [b_i - 1/2, b_i + 1/2]|.
// Every thread owns a column of K voxels along z and walks the views (the
// forward scatter picks the column per view, see sf_fwd_kernel); per
// voxel-view it visits the footprint's pixel window (clipped to the
// detector).  The forward projection scatters a_ij mu_j (through LDS tiles whose
// pixels are added to the image with FP32 atomics);
// the back-projection and both gradients gather, so they are deterministic.
//
// Forward gradient: s_j = sum_i a_ij dL/dl_i, then the ray kernel's nine
// sums B_c = sum s_j G_c(j), T_ac = sum s_j (I_a - centre_a) G_c(j) with the
// central-difference gradient in index units; the ray kernel's FP64
// finalize turns them into dL/dtheta.
// Back-projection gradient: d_j = sum_i a_ij (l_a, l_b)_i (central
// differences at the pixel centres), then the voxel kernel's twelve sums
// with c = (d_a, d_b, -(d_a a' + d_b b')) e_j / w' (a', b', w' of the voxel
// centre), finalized by the voxel kernel's FP64 finalize.
#include <cmath>

#include "dp_internal.h"

namespace dp {

constexpr int kSfBx = 64, kSfBy = 4, kSfCol = 8;
constexpr int kFpSF = DP_FP_SF, kFpDD = DP_FP_DD;

// Footprint of one voxel in one view, in FP32 pixel coordinates relative
// to an integer base pixel (abase, bbase), so that breakpoints of magnitude
// ~1e3 pixels keep ~1e-6 pixel resolution.
struct SfFootprint {
    float tau[4];     // trapezoid breakpoints (column), relative to abase
    float r01, r23;   // 1 / (2 (tau1 - tau0)), 1 / (2 (tau3 - tau2)); 0 for a vertical edge
    float blo, bhi;   // row rectangle, relative to bbase
    float L;          // amplitude
    int abase, bbase;
    int a0, a1, b0, b1;  // pixel window (inclusive, absolute), clipped; empty if a0 > a1 or b0 > b1
};

constexpr double kSfPixClamp = 1048576.0;  // projections beyond 2^20 pixels are off any detector

// Integral of the unit-height trapezoid over [x0, x1] (relative to abase),
// segment by segment: rising edge (x - t0) / (t1 - t0), plateau, falling
// edge (t3 - x) / (t3 - t2).  Each term is a product of short differences,
// so no digits are lost when breakpoints lie far from the cell; an edge the
// cell does not reach (or a vertical one) contributes exactly zero.
template <int KIND>
__device__ inline float trap_integral(float x0, float x1, const SfFootprint& f)
{
    const float* t = f.tau;
    float s = fmaxf(fminf(x1, t[2]) - fmaxf(x0, t[1]), 0.0f);
    if (KIND == kFpSF) {
        const float l0 = fmaxf(x0, t[0]), r0 = fminf(x1, t[1]);
        s += fmaxf(r0 - l0, 0.0f) * ((r0 - t[0]) + (l0 - t[0])) * f.r01;
        const float l1 = fmaxf(x0, t[2]), r1 = fminf(x1, t[3]);
        s += fmaxf(r1 - l1, 0.0f) * ((t[3] - l1) + (t[3] - r1)) * f.r23;
    }
    return s;
}

__device__ inline float row_overlap(float b, float lo, float hi)
{
    const float o = fminf(b + 0.5f, hi) - fmaxf(b - 0.5f, lo);
    return o > 0.0f ? o : 0.0f;
}

// Slope factor of an edge from lo to hi, 1 / (2 (hi - lo)), to ~1 ulp (hardware
// rcp: only relative precision is needed).  An edge narrower than 1e-30 pixels
// counts as vertical, so the factor is finite.
__device__ inline float sf_slope(float lo, float hi)
{
    return hi - lo > 1.0e-30f ? 0.5f * __builtin_amdgcn_rcpf(hi - lo) : 0.0f;
}

// Slopes and pixel window of a footprint whose breakpoints, rows and bases are
// set (the bases and relative offsets are bounded, so no overflow).
__device__ inline void sf_window(const GeoScalars& s, SfFootprint& f)
{
    f.r01 = sf_slope(f.tau[0], f.tau[1]);
    f.r23 = sf_slope(f.tau[2], f.tau[3]);
    f.a0 = max(f.abase + (int)floorf(f.tau[0] - 0.5f) + 1, 0);
    f.a1 = min(f.abase + (int)ceilf(f.tau[3] + 0.5f) - 1, s.nu - 1);
    f.b0 = max(f.bbase + (int)floorf(f.blo - 0.5f) + 1, 0);
    f.b1 = min(f.bbase + (int)ceilf(f.bhi + 0.5f) - 1, s.nv - 1);
}

// The parts every producer shares: sort (SF), slopes, amplitude, window.
// t: column breakpoints (SF: four corners; DD: the two boundaries in t[0],
// t[1]), bb: the two row bounds, both relative to the bases; d: the line
// from the source to the voxel centre (mm).
template <int KIND>
__device__ inline void sf_finish(const GeoScalars& s, int dom, float* t, const float* bb,
                                 const float* d, int abase, int bbase, SfFootprint& f)
{
    if (KIND == kFpSF) {
#define DP_CX(p, q)                                                  \
    {                                                                \
        const float lo_ = fminf(t[p], t[q]), hi_ = fmaxf(t[p], t[q]); \
        t[p] = lo_;                                                  \
        t[q] = hi_;                                                  \
    }
        DP_CX(0, 1) DP_CX(2, 3) DP_CX(0, 2) DP_CX(1, 3) DP_CX(1, 2)
#undef DP_CX
    } else {
        const float lo = fminf(t[0], t[1]), hi = fmaxf(t[0], t[1]);
        t[0] = t[1] = lo;
        t[2] = t[3] = hi;
    }
    for (int c = 0; c < 4; ++c) f.tau[c] = t[c];
    f.blo = fminf(bb[0], bb[1]);
    f.bhi = fmaxf(bb[0], bb[1]);
    // amplitude: SF the chord min_a h_a |d| / |d_a|, DD the slab path
    // h_dom |d| / |d_dom|; it scales the weights, so FP32 is enough
    const float h[3] = {(float)s.vx, (float)s.vy, (float)s.vz};
    const float n = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    float L;
    if (KIND == kFpSF) {
        L = INFINITY;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (d[c] != 0.0f) L = fminf(L, h[c] * n * __builtin_amdgcn_rcpf(fabsf(d[c])));
    } else {
        L = d[dom] != 0.0f ? h[dom] * n * __builtin_amdgcn_rcpf(fabsf(d[dom])) : 0.0f;
    }
    f.L = L;
    f.abase = abase;
    f.bbase = bbase;
    sf_window(s, f);
}

// Column breakpoint line q of voxel column (i, j): SF corner (i +- 1/2,
// j +- 1/2), DD boundary across the non-dominant transaxial axis.
template <int KIND>
__device__ inline void sf_line(int q, int dom, double& dx, double& dy)
{
    if (KIND == kFpSF) {
        dx = (q & 1) ? 0.5 : -0.5;
        dy = (q & 2) ? 0.5 : -0.5;
    } else {
        const double off = q ? 0.5 : -0.5;
        dx = dom == 0 ? 0.0 : off;  // dom x: boundaries across y
        dy = dom == 0 ? off : 0.0;
    }
}

// Per-voxel FP64 footprint of voxel (i, j, k) in view g; false if any
// projected point lies at or behind the source plane.  src: the source in
// object-frame index units; dom: DD's dominant axis of the view.
template <int KIND>
__device__ inline bool sf_footprint(const ViewGeo& g, const GeoScalars& s, const double* src,
                                    int dom, int i, int j, int k, SfFootprint& f)
{
    const double fi = i, fj = j, fk = k;
    const double U0 = fma(g.PUd[0], fi, fma(g.PUd[1], fj, fma(g.PUd[2], fk, g.PUd[3])));
    const double V0 = fma(g.PVd[0], fi, fma(g.PVd[1], fj, fma(g.PVd[2], fk, g.PVd[3])));
    const double W0 = fma(g.PWd[0], fi, fma(g.PWd[1], fj, fma(g.PWd[2], fk, g.PWd[3])));
    constexpr int NL = KIND == kFpSF ? 4 : 2;
    double td[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        double dx, dy;
        sf_line<KIND>(q, dom, dx, dy);
        const double U = fma(g.PUd[0], dx, fma(g.PUd[1], dy, U0));
        const double W = fma(g.PWd[0], dx, fma(g.PWd[1], dy, W0));
        if (!(W > 0.0)) return false;
        td[q] = fmin(fmax(U / W + s.cu, -kSfPixClamp), kSfPixClamp);
    }
    double bd[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const double dz = c ? 0.5 : -0.5;
        const double V = fma(g.PVd[2], dz, V0), W = fma(g.PWd[2], dz, W0);
        if (!(W > 0.0)) return false;
        bd[c] = fmin(fmax(V / W + s.cv, -kSfPixClamp), kSfPixClamp);
    }
    const double ab = floor(td[0]), bbv = floor(bd[0]);
    float t[4], bb[2];
#pragma unroll
    for (int q = 0; q < NL; ++q) t[q] = (float)(td[q] - ab);
    bb[0] = (float)(bd[0] - bbv);
    bb[1] = (float)(bd[1] - bbv);
    const float d[3] = {(float)((fi - src[0]) * s.vx), (float)((fj - src[1]) * s.vy),
                        (float)((fk - src[2]) * s.vz)};
    sf_finish<KIND>(s, dom, t, bb, d, (int)ab, (int)bbv, f);
    return true;
}

// FP64 anchors of voxel column (i, j) at height ka for one view.  Along the
// column each breakpoint line and the centre line move only in z, so with
// U(dk) = U0 + dk P_uz and W(dk) = W0 + dk P_wz the projection is exactly
//   U(dk) / W(dk) = U0 / W0 + dk N / W(dk),   N = (P_uz W0 - P_wz U0) / W0,
// and only the small offset dk N / W(dk) is evaluated per voxel, in FP32.
struct SfColumn {
    bool fast;       // false: an anchor within 1 mm of the source plane (per-voxel FP64)
    bool front;      // fast, and every line stays in front of the source along the column
    int abase, bbase;
    float tfr[4], tn[4], tw[4];  // breakpoint lines: anchor offset from abase, N, W0
    float bfr, bn, bw;           // centre line: row offset from bbase, N_v, W0
    float ucfr, ucn;             // centre line: column offset from abase, N_u
    float uco, bco;              // abase - c_u, bbase - c_v (offsets from the detector centre)
    float pwz, ka;
    float d0, d1, d2o;           // source-to-voxel line: x, y (mm) and z offset
    float i0, i1;                // 1 / |d0|, 1 / |d1|
};

template <int KIND>
__device__ inline SfColumn sf_column(const ViewGeo& g, const GeoScalars& s, const double* src,
                                     int dom, int i, int j, int ka)
{
    SfColumn c;
    c.fast = c.front = false;
    const double fi = i, fj = j, fk = ka;
    constexpr int NL = KIND == kFpSF ? 4 : 2;
    double A[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        double dx, dy;
        sf_line<KIND>(q, dom, dx, dy);
        const double U = fma(g.PUd[0], fi + dx, fma(g.PUd[1], fj + dy, fma(g.PUd[2], fk, g.PUd[3])));
        const double W = fma(g.PWd[0], fi + dx, fma(g.PWd[1], fj + dy, fma(g.PWd[2], fk, g.PWd[3])));
        if (!(W >= 1.0)) return c;
        const double iw = 1.0 / W;
        A[q] = fmin(fmax(U * iw + s.cu, -kSfPixClamp), kSfPixClamp);
        c.tn[q] = (float)((g.PUd[2] * W - g.PWd[2] * U) * iw);
        c.tw[q] = (float)W;
    }
    const double Uc = fma(g.PUd[0], fi, fma(g.PUd[1], fj, fma(g.PUd[2], fk, g.PUd[3])));
    const double V = fma(g.PVd[0], fi, fma(g.PVd[1], fj, fma(g.PVd[2], fk, g.PVd[3])));
    const double W = fma(g.PWd[0], fi, fma(g.PWd[1], fj, fma(g.PWd[2], fk, g.PWd[3])));
    if (!(W >= 1.0)) return c;
    const double iw = 1.0 / W;
    const double B = fmin(fmax(V * iw + s.cv, -kSfPixClamp), kSfPixClamp);
    const double Ac = fmin(fmax(Uc * iw + s.cu, -kSfPixClamp), kSfPixClamp);
    c.bn = (float)((g.PVd[2] * W - g.PWd[2] * V) * iw);
    c.ucn = (float)((g.PUd[2] * W - g.PWd[2] * Uc) * iw);
    c.bw = (float)W;
    const double ab = floor(A[0]), bb = floor(B);
    c.abase = (int)ab;
    c.bbase = (int)bb;
#pragma unroll
    for (int q = 0; q < NL; ++q) c.tfr[q] = (float)(A[q] - ab);
    c.bfr = (float)(B - bb);
    c.ucfr = (float)(Ac - ab);
    c.uco = (float)(ab - s.cu);
    c.bco = (float)(bb - s.cv);
    c.pwz = (float)g.PWd[2];
    c.ka = (float)ka;
    c.d0 = (float)((fi - src[0]) * s.vx);
    c.d1 = (float)((fj - src[1]) * s.vy);
    c.d2o = (float)(-src[2] * s.vz);
    c.i0 = __builtin_amdgcn_rcpf(fabsf(c.d0));
    c.i1 = __builtin_amdgcn_rcpf(fabsf(c.d1));
    c.fast = true;
    // depths are linear along the column: positive at both ends, positive between
    const float e0 = -0.5f * kSfCol - 0.5f, e1 = 0.5f * kSfCol - 0.5f;
    float wmin = fminf(fmaf(e0, c.pwz, c.bw), fmaf(e1, c.pwz, c.bw));
#pragma unroll
    for (int q = 0; q < NL; ++q)
        wmin = fminf(wmin, fminf(fmaf(e0, c.pwz, c.tw[q]), fmaf(e1, c.pwz, c.tw[q])));
    c.front = wmin > 0.0f;
    return c;
}

// Footprint of voxel (i, j, k) from its column's anchors (FP32), falling
// back to the per-voxel FP64 footprint when the column has no safe anchor.
template <int KIND>
__device__ inline bool sf_voxel(const SfColumn& c, const ViewGeo& g, const GeoScalars& s,
                                const double* src, int dom, int i, int j, int k, SfFootprint& f)
{
    if (!c.fast) return sf_footprint<KIND>(g, s, src, dom, i, j, k, f);
    constexpr int NL = KIND == kFpSF ? 4 : 2;
    const float dk = (float)k - c.ka;
    float t[4] = {0.f, 0.f, 0.f, 0.f}, bb[2];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const float W = fmaf(dk, c.pwz, c.tw[q]);
        if (!(W > 0.0f)) return false;
        t[q] = fmaf(dk * c.tn[q], __builtin_amdgcn_rcpf(W), c.tfr[q]);  // offset <~ 10 px
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float dz = dk + (e ? 0.5f : -0.5f);
        const float W = fmaf(dz, c.pwz, c.bw);
        if (!(W > 0.0f)) return false;
        bb[e] = fmaf(dz * c.bn, __builtin_amdgcn_rcpf(W), c.bfr);
    }
    const float d[3] = {c.d0, c.d1, fmaf((float)k, (float)s.vz, c.d2o)};
    sf_finish<KIND>(s, dom, t, bb, d, c.abase, c.bbase, f);
    return true;
}

// Projected row (relative to bbase) of the column's centre line at dk voxels
// from the anchor; a front column only.
__device__ inline float sf_row(const SfColumn& c, float dk)
{
    return fmaf(dk * c.bn, __builtin_amdgcn_rcpf(fmaf(dk, c.pwz, c.bw)), c.bfr);
}

// Correctly rounded square root of a normal x up to rare last bits, in half
// the instructions of sqrtf (no scaling of denormals).
__device__ inline float sf_sqrt(float x)
{
    const float y = __builtin_amdgcn_rsqf(x), r = x * y;
    return fmaf(fmaf(-r, r, x), 0.5f * y, r);
}

// Footprint of voxel k of a front column, without its pixel window: no depth
// tests, and the row bound shared with the voxel below (row_lo, updated to the
// bound shared with the next one).
template <int KIND>
struct SfBox {
    float t[4];      // breakpoints in order (DD: t[0] = t[1], t[2] = t[3])
    float blo, bhi;  // row rectangle
    float L;         // amplitude
};

template <int KIND>
__device__ inline SfBox<KIND> sf_box(const SfColumn& c, const GeoScalars& s, int dom, int k,
                                     float& row_lo)
{
    constexpr int NL = KIND == kFpSF ? 4 : 2;
    SfBox<KIND> f;
    const float dk = (float)k - c.ka;
    float t[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q)
        t[q] = fmaf(dk * c.tn[q], __builtin_amdgcn_rcpf(fmaf(dk, c.pwz, c.tw[q])), c.tfr[q]);
    const float h0 = (float)s.vx, h1 = (float)s.vy, h2 = (float)s.vz;
    const float d2 = fmaf((float)k, h2, c.d2o);
    const float n = sf_sqrt(c.d0 * c.d0 + c.d1 * c.d1 + d2 * d2);
    if constexpr (KIND == kFpSF) {
        const float l0 = fminf(t[0], t[1]), g0 = fmaxf(t[0], t[1]);
        const float l1 = fminf(t[2], t[3]), g1 = fmaxf(t[2], t[3]);
        f.t[0] = fminf(l0, l1);
        f.t[3] = fmaxf(g0, g1);
        const float m0 = fmaxf(l0, l1), m1 = fminf(g0, g1);
        f.t[1] = fminf(m0, m1);
        f.t[2] = fmaxf(m0, m1);
        // an axis the line does not move along has 1 / |d| = inf and drops out
        f.L = fminf(fminf(h0 * n * c.i0, h1 * n * c.i1),
                    h2 * n * __builtin_amdgcn_rcpf(fabsf(d2)));
    } else {
        f.t[0] = f.t[1] = fminf(t[0], t[1]);
        f.t[2] = f.t[3] = fmaxf(t[0], t[1]);
        const float hd = dom == 0 ? h0 : h1, dd = dom == 0 ? c.d0 : c.d1, id = dom == 0 ? c.i0 : c.i1;
        f.L = dd != 0.0f ? hd * n * id : 0.0f;
    }
    const float up = sf_row(c, dk + 0.5f);
    f.blo = fminf(row_lo, up);
    f.bhi = fmaxf(row_lo, up);
    row_lo = up;
    return f;
}

// The same voxel with its slopes and window, for the general pixel loops.
template <int KIND>
__device__ inline void sf_unbox(const SfBox<KIND>& x, const SfColumn& c, const GeoScalars& s,
                                SfFootprint& f)
{
    for (int q = 0; q < 4; ++q) f.tau[q] = x.t[q];
    f.blo = x.blo;
    f.bhi = x.bhi;
    f.L = x.L;
    f.abase = c.abase;
    f.bbase = c.bbase;
    sf_window(s, f);
}

// Source position in object-frame (unpadded) voxel-index units, and the
// view's dominant transaxial axis for DD (0 = x, 1 = y).
__device__ inline int sf_source(const ViewGeo& g, const GeoScalars& s, double* src)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) src[c] = g.OT[c] - kPadV - s.sad * g.EW[c];
    const double ox = (src[0] - 0.5 * (s.nx - 1)) * s.vx, oy = (src[1] - 0.5 * (s.ny - 1)) * s.vy;
    return fabs(ox) >= fabs(oy) ? 0 : 1;
}

// The footprint's pixels column by column: fn(a, b, w) for every pixel of
// the window with a non-zero weight w = column integral x row overlap
// (without the amplitude L); the column integral is evaluated once per
// column.
template <int KIND, typename Fn>
__device__ inline void sf_for_each(const SfFootprint& f, Fn&& fn)
{
    for (int a = f.a0; a <= f.a1; ++a) {
        const float x = (float)(a - f.abase);
        const float wa = trap_integral<KIND>(x - 0.5f, x + 0.5f, f);
        if (wa == 0.0f) continue;
        for (int b = f.b0; b <= f.b1; ++b) {
            const float wb = row_overlap((float)(b - f.bbase), f.blo, f.bhi);
            if (wb != 0.0f) fn(a, b, wa * wb);
        }
    }
}

// ---------------------------------------------------------------------------
// Gathers.  Bound by VALU issue, not by the loads: a voxel's window is read as
// a patch of up to 4 columns and 3 rows (nearly every footprint: a voxel
// magnified to about two pixels), one unaligned 16-byte load per row and
// channel, and every weight of the patch is formed without branches from
// cell edges clamped to the footprint's segments (each edge serves both its
// cells; cells outside get exactly zero).  Columns 2, 3 and row 2 are skipped
// when no lane of the wavefront has them.  Wavefronts with larger windows
// take their pixels in several such quads of up to 5 rows, and lanes beyond
// that, or whose sum is not finite (a pixel of weight zero may hold
// anything), pixel by pixel.  All of these add the same products in the same
// order (columns outside, rows inside).
// Measured from a 256^3 volume of 0.8 mm voxels and 384^2 views of 0.8 mm
// pixels, against loops over each lane's own window in an unrolled column:
// DD back-projection of 64 views 9.88 -> 3.79 ms (2.8e11 voxel-view updates/s,
// about 110 VALU instructions each beside the FP64 column anchors) and its
// gradient 5.40 -> 2.18 ms; SF forward gradient of 4 views 0.78 -> 0.30 ms.  VALU
// busy 130, 47 and 97 % of the 4-cycle model (the back-projection gradient's
// volume is mostly zero there), texture addresser 55, 27 and 34 %.
// Four blocks per CU; five or six spill and are slower (1.03x, 1.4x).
// ---------------------------------------------------------------------------

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) const f32x4u sf_global4;
typedef __attribute__((address_space(1))) const char sf_bytes;

__device__ inline bool sf_any(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; }

// floor(x) as an integer in one instruction (saturating; 0 for NaN).
__device__ inline int sf_floor(float x)
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// A detector image [nv][nu] (at most 16384 x 16384: 32-bit byte offsets from a
// wave-uniform base).
struct SfImage {
    static constexpr int C = 1;
    const float* img;
    int nu;
    __device__ inline void row4(int a, int b, float (&v)[1][4]) const
    {
        const unsigned o = (unsigned)(__mul24(b, 4 * nu) + 4 * a);
        const f32x4u q = *(sf_global4*)((sf_bytes*)img + o);
        v[0][0] = q.x; v[0][1] = q.y; v[0][2] = q.z; v[0][3] = q.w;
    }
    __device__ inline void pixel(int a, int b, float (&v)[1]) const { v[0] = img[(unsigned)(b * nu + a)]; }
};

// A detector gradient image: (dl/da, dl/db) per pixel, [nv][nu].
struct SfGradImage {
    static constexpr int C = 2;
    const float2* img;
    int nu;
    __device__ inline void row4(int a, int b, float (&v)[2][4]) const
    {
        const unsigned o = (unsigned)(__mul24(b, 8 * nu) + 8 * a);
        const f32x4u q = *(sf_global4*)((sf_bytes*)img + o), r = *(sf_global4*)((sf_bytes*)img + 16 + o);
        v[0][0] = q.x; v[1][0] = q.y; v[0][1] = q.z; v[1][1] = q.w;
        v[0][2] = r.x; v[1][2] = r.y; v[0][3] = r.z; v[1][3] = r.w;
    }
    __device__ inline void pixel(int a, int b, float (&v)[2]) const
    {
        const float2 q = img[(unsigned)(b * nu + a)];
        v[0] = q.x; v[1] = q.y;
    }
};

// Adds the pixels of the window's columns a .. a + 3 (a >= 0, nu >= 4) and
// first 5 rows.  The loads start at most at column nu - 4; columns before a
// are left out.
template <int KIND, class Img>
__device__ inline void sf_quad(const SfFootprint& f, const GeoScalars& s, const Img& img, int a,
                               float (&acc)[Img::C])
{
    constexpr int NR = 5;
    const int s0 = min(a, s.nu - 4);
    const float x = (float)(s0 - f.abase);
    float v[NR][Img::C][4], wb[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        img.row4(s0, min(f.b0 + r, s.nv - 1), v[r]);
        wb[r] = f.b0 + r <= f.b1 ? row_overlap((float)(f.b0 + r - f.bbase), f.blo, f.bhi) : 0.0f;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float wa = s0 + t >= a ? trap_integral<KIND>(x + (float)t - 0.5f, x + (float)t + 0.5f, f)
                                     : 0.0f;
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int c = 0; c < Img::C; ++c) acc[c] = fmaf(wa * wb[r], v[r][c][t], acc[c]);
    }
}

// acc = sum_i a_ij img_i over the footprint, any window.
template <int KIND, class Img>
__device__ inline void sf_gather(const SfFootprint& f, const GeoScalars& s, const Img& img,
                                 float (&acc)[Img::C])
{
#pragma unroll
    for (int c = 0; c < Img::C; ++c) acc[c] = 0.0f;
    bool loop = s.nu < 4 || f.b1 - f.b0 >= 5;
    if (!loop && f.b0 <= f.b1)
        for (int a = f.a0; a <= f.a1; a += 4) sf_quad<KIND>(f, s, img, a, acc);
#pragma unroll
    for (int c = 0; c < Img::C; ++c) loop = loop || !(fabsf(acc[c]) < INFINITY);
    if (loop) {
#pragma unroll
        for (int c = 0; c < Img::C; ++c) acc[c] = 0.0f;
        sf_for_each<KIND>(f, [&](int a, int b, float w) {
            float v[Img::C];
            img.pixel(a, b, v);
#pragma unroll
            for (int c = 0; c < Img::C; ++c) acc[c] = fmaf(w, v[c], acc[c]);
        });
    }
#pragma unroll
    for (int c = 0; c < Img::C; ++c) acc[c] *= f.L;
}

// Weights of N cells from edge e on (cells [e, e + 1], ...): column integrals
// of the trapezoid, row overlaps.
template <int KIND, int N>
__device__ inline void sf_cells(const float (&t)[4], float e, float (&w)[N])
{
    if constexpr (KIND == kFpSF) {
        const float r01 = sf_slope(t[0], t[1]), r23 = sf_slope(t[2], t[3]);
        float p = __builtin_amdgcn_fmed3f(e, t[1], t[2]);
        float u = __builtin_amdgcn_fmed3f(e, t[0], t[1]), du = u - t[0];
        float d = __builtin_amdgcn_fmed3f(e, t[2], t[3]), dd = t[3] - d;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const float x = e + (float)(q + 1);
            const float p1 = __builtin_amdgcn_fmed3f(x, t[1], t[2]);
            const float u1 = __builtin_amdgcn_fmed3f(x, t[0], t[1]), du1 = u1 - t[0];
            const float d1 = __builtin_amdgcn_fmed3f(x, t[2], t[3]), dd1 = t[3] - d1;
            w[q] = fmaf((d1 - d) * (dd + dd1), r23, fmaf((u1 - u) * (du1 + du), r01, p1 - p));
            p = p1; u = u1; du = du1; d = d1; dd = dd1;
        }
    } else {
        float p = __builtin_amdgcn_fmed3f(e, t[0], t[3]);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const float p1 = __builtin_amdgcn_fmed3f(e + (float)(q + 1), t[0], t[3]);
            w[q] = p1 - p;
            p = p1;
        }
    }
}

// The gather of a front column's voxel (nu >= 4).
template <int KIND, class Img>
__device__ inline void sf_gather_box(const SfBox<KIND>& x, const SfColumn& c, const GeoScalars& s,
                                     const Img& img, float (&acc)[Img::C])
{
    const int a0 = max(c.abase + sf_floor(x.t[0] - 0.5f) + 1, 0), s0 = min(a0, s.nu - 4);
    const int b0 = max(c.bbase + sf_floor(x.blo - 0.5f) + 1, 0);
    const float xs = (float)(s0 - c.abase), ys = (float)(b0 - c.bbase);
    const float ta = x.t[3] + 0.5f, tb = x.bhi + 0.5f;
    const bool fits = (ta <= xs + 4.0f || s0 + 4 >= s.nu) && (tb <= ys + 3.0f || b0 + 3 >= s.nv);
    bool general = true;
    if (!sf_any(!fits)) {
        float v[3][Img::C][4], wa[4], wb[3];
        const bool row2 = sf_any(tb > ys + 2.0f);
        img.row4(s0, min(b0, s.nv - 1), v[0]);
        img.row4(s0, min(b0 + 1, s.nv - 1), v[1]);
        if (row2) img.row4(s0, min(b0 + 2, s.nv - 1), v[2]);
        const float tr[4] = {x.blo, x.blo, x.bhi, x.bhi};
        sf_cells<kFpDD, 3>(tr, ys - 0.5f, wb);
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (b0 + r >= s.nv) wb[r] = 0.0f;
        sf_cells<KIND, 4>(x.t, xs - 0.5f, wa);
#pragma unroll
        for (int q = 0; q < Img::C; ++q) acc[q] = 0.0f;
        const auto add = [&](int t) {
#pragma unroll
            for (int q = 0; q < Img::C; ++q) {
                acc[q] = fmaf(wa[t] * wb[0], v[0][q][t], acc[q]);
                acc[q] = fmaf(wa[t] * wb[1], v[1][q][t], acc[q]);
                if (row2) acc[q] = fmaf(wa[t] * wb[2], v[2][q][t], acc[q]);
            }
        };
        add(0);
        add(1);
        if (sf_any(ta > xs + 2.0f)) add(2);
        if (sf_any(ta > xs + 3.0f)) add(3);
        general = false;
#pragma unroll
        for (int q = 0; q < Img::C; ++q) {
            general = general || !(fabsf(acc[q]) < INFINITY);
            acc[q] *= x.L;
        }
    }
    if (general) {
        SfFootprint f;
        sf_unbox<KIND>(x, c, s, f);
        sf_gather<KIND>(f, s, img, acc);
    }
}

// Walks the nk voxels from kb on of a thread's column in one view, calling
// fn(kk, k, acc) with the footprint-weighted image sums of every projected
// voxel for which want(kk) holds.  Wavefronts whose columns all lie in front
// of the source take the fast gather; the voxel loop stays rolled (one copy of
// the code, and of its registers).
template <int KIND, class Img, class Want, class Fn>
__device__ inline void sf_walk(const SfColumn& col, const ViewGeo& g, const GeoScalars& s,
                               const double* src, int dom, int i, int j, int kb, int nk,
                               const Img& img, Want&& want, Fn&& fn)
{
    if (s.nu >= 4 && !sf_any(!col.front)) {
        float row_lo = sf_row(col, (float)kb - col.ka - 0.5f);
#pragma unroll 1
        for (int kk = 0; kk < nk; ++kk) {
            const SfBox<KIND> x = sf_box<KIND>(col, s, dom, kb + kk, row_lo);
            if (!want(kk)) continue;
            float acc[Img::C];
            sf_gather_box<KIND>(x, col, s, img, acc);
            fn(kk, kb + kk, acc);
        }
    } else {
#pragma unroll 1
        for (int kk = 0; kk < nk; ++kk) {
            if (!want(kk)) continue;
            SfFootprint f;
            if (!sf_voxel<KIND>(col, g, s, src, dom, i, j, kb + kk, f)) continue;
            float acc[Img::C];
            sf_gather<KIND>(f, s, img, acc);
            fn(kk, kb + kk, acc);
        }
    }
}

// ---------------------------------------------------------------------------
// Forward scatter.  A wavefront's 64 lanes take 64 neighbouring voxels across
// the view's rays, not along them: lanes along y when the rays run closest to
// the x axis (DD's dominant axis 0), along x otherwise, so their footprints
// cover neighbouring pixels instead of all landing on the same ones.
// Each wavefront projects a brick of one view on its own: 64 voxels across,
// `steps` along the rays, kSfCol along z (or a part of them).  The footprints
// add up in the wavefront's own LDS tile, the rectangle of pixels that the
// brick projects onto, and each of those pixels goes to memory with one FP32
// atomic.  The tile takes plain reads and writes, one window column of all
// lanes at a time: lanes whose windows start in different detector columns
// cannot meet in a pixel then, and LDS operations of a wavefront are carried
// out in order.  Lanes that do start in the same column (voxels narrower than a pixel)
// take turns.
// Voxels with wider windows, and those that hold no number, go to memory pixel by pixel.
// FP32 atomics are what this avoids: straight to memory, one per pixel of
// every footprint, they took most of the kernel's time, and LDS ones take
// about 110 cycles per wavefront (measured: ds_add_f32, no conflicts).  What is
// left is the chain of each column's read, add and write: VALU busy 53 % of the
// 4-cycle model, texture addresser 34 %, LDS conflicts 2 % of cycles.
// ---------------------------------------------------------------------------

// Voxels along the rays per brick, and tile pixels per wavefront (four blocks,
// 16 wavefronts, per CU).  SF, 4 views of 384^2 from 256^3: 0.47 ms; 1 / 4 / 8
// voxels 0.56 / 0.52 / 0.58, tiles of 1600 / 4092 pixels 0.48 / 0.73 ms.
constexpr int kSfSteps = 2;
constexpr int kSfTile = 2496;
constexpr int kSfFwdWaves = 4096;    // one voxel along the rays if there are fewer bricks than this
constexpr int kSfPatchCols = 4;
constexpr int kSfQuads = 4;          // patches per axis of the largest window added to a tile

struct SfRect {
    int a0, b0, w, h;  // pixels [a0, a0 + w) x [b0, b0 + h); empty if w h = 0
    bool known;        // false: the brick reaches within 1 mm of the source plane
};

// Pixels that the voxels [i0, i1] x [j0, j1] x [k0, k1] project onto: their
// footprints lie in the hull of the projections of the brick's corners if all
// of them are at least 1 mm in front of the source.  Wave-uniform; every
// eight lanes take the eight corners.
__device__ inline SfRect sf_rect(const ViewGeo& g, const GeoScalars& s, int i0, int i1, int j0,
                                 int j1, int k0, int k1)
{
    const int q = threadIdx.x & 7;
    const double ci = (q & 1) ? i1 + 0.5 : i0 - 0.5, cj = (q & 2) ? j1 + 0.5 : j0 - 0.5;
    const double ck = (q & 4) ? k1 + 0.5 : k0 - 0.5;
    const double U = fma(g.PUd[0], ci, fma(g.PUd[1], cj, fma(g.PUd[2], ck, g.PUd[3])));
    const double V = fma(g.PVd[0], ci, fma(g.PVd[1], cj, fma(g.PVd[2], ck, g.PVd[3])));
    const double W = fma(g.PWd[0], ci, fma(g.PWd[1], cj, fma(g.PWd[2], ck, g.PWd[3])));
    const bool front = W >= 1.0;
    const double iw = front ? 1.0 / W : 0.0;
    float amin = (float)fmin(fmax(U * iw + s.cu, -4.0), s.nu + 3.0), amax = amin;
    float bmin = (float)fmin(fmax(V * iw + s.cv, -4.0), s.nv + 3.0), bmax = bmin;
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) {
        amin = fminf(amin, __shfl_xor(amin, off));
        amax = fmaxf(amax, __shfl_xor(amax, off));
        bmin = fminf(bmin, __shfl_xor(bmin, off));
        bmax = fmaxf(bmax, __shfl_xor(bmax, off));
    }
    SfRect r;
    // cells overlapping the hull, with a margin for rounding
    const int a0 = max(0, (int)floorf(amin - 0.52f) + 1), a1 = min(s.nu - 1, (int)ceilf(amax + 0.52f) - 1);
    const int b0 = max(0, (int)floorf(bmin - 0.52f) + 1), b1 = min(s.nv - 1, (int)ceilf(bmax + 0.52f) - 1);
    r.a0 = __builtin_amdgcn_readfirstlane(a0);
    r.b0 = __builtin_amdgcn_readfirstlane(b0);
    r.w = __builtin_amdgcn_readfirstlane(max(0, a1 - a0 + 1));
    r.h = __builtin_amdgcn_readfirstlane(max(0, b1 - b0 + 1));
    r.known = !sf_any(!front);
    return r;
}

// One step's front columns (nu >= 4; lanes with p beyond the volume hold
// active = false) into the wavefront's tile, whose cells from npix on are
// a dump for rows outside it.
template <int KIND>
__device__ inline void sf_scatter(const SfColumn& c, const GeoScalars& s, int dom, int kb, int nk,
                                  const float* __restrict__ mu, size_t plane, bool active,
                                  const SfRect& rect, float* tile, float* __restrict__ img)
{
    const int npix = rect.w * rect.h, lane = threadIdx.x;
    float row_lo = sf_row(c, (float)kb - c.ka - 0.5f);
    float next = active ? mu[0] : 0.0f;
#pragma unroll 1
    for (int kk = 0; kk < nk; ++kk) {
        const float m = next;
        next = active && kk + 1 < nk ? mu[(size_t)(kk + 1) * plane] : 0.0f;
        const SfBox<KIND> x = sf_box<KIND>(c, s, dom, kb + kk, row_lo);
        if (!sf_any(m != 0.0f)) continue;
        const float ta = x.t[3] + 0.5f, tb = x.bhi + 0.5f, scale = x.L * m;
        // window, not clipped: first column and row relative to the bases
        const int ra = sf_floor(x.t[0] - 0.5f) + 1, rb = sf_floor(x.blo - 0.5f) + 1;
        const float xs = (float)ra - 0.5f, ys = (float)rb - 0.5f;
        // (a patch also adds to pixels of weight zero, where inf and NaN must not go)
        const bool fits = ta <= xs + (0.5f + 4 * kSfQuads) && tb <= ys + (0.5f + 3 * kSfQuads) &&
                          fabsf(scale) < INFINITY;
        // lanes `turns` apart start in different columns
        const int pa = c.abase + ra;
        int turns = 1;
        for (; turns < 64; turns *= 2) {
            const int d = pa - __shfl_up(pa, turns);
            if (!sf_any(lane >= turns && active && d <= 0) || !sf_any(lane >= turns && active && d >= 0))
                break;
        }
        const float tr[4] = {x.blo, x.blo, x.bhi, x.bhi};
        const bool mine = m != 0.0f && fits;
        // adds the window's patch of 4 columns and 3 rows from (xh, ye) on
        const auto patch = [&](float xh, int ca, float ye, int cb) {
            const bool row2 = sf_any(tb > ye + 2.5f), col2 = sf_any(ta > xh + 2.5f),
                       col3 = sf_any(ta > xh + 3.5f);
            float wa[4], wb[3];
            float* row[3];
            sf_cells<KIND, 4>(x.t, xh, wa);
            sf_cells<kFpDD, 3>(tr, ye, wb);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                row[r] = tile + ((unsigned)(cb + r) < (unsigned)rect.h ? __mul24(cb + r, rect.w) + ca : npix);
                wb[r] *= scale;
            }
            for (int turn = 0; turn < turns; ++turn) {
                const bool now = mine && (lane & (turns - 1)) == turn;
#pragma unroll
                for (int t = 0; t < kSfPatchCols; ++t) {
                    if ((t == 2 && !col2) || (t == 3 && !col3)) break;
                    // the column's reads follow the previous one's writes
                    __builtin_amdgcn_wave_barrier();
                    asm volatile("" ::: "memory");
                    if (now && (unsigned)(ca + t) < (unsigned)rect.w) {
                        float* r0 = row[0] + t;
                        float* r1 = row[1] + t;
                        float* r2 = row[2] + t;
                        const float v0 = *r0, v1 = *r1;
                        if (row2) {
                            const float v2 = *r2;
                            *r2 = fmaf(wa[t], wb[2], v2);
                        }
                        *r0 = fmaf(wa[t], wb[0], v0);
                        *r1 = fmaf(wa[t], wb[1], v1);
                    }
                }
            }
        };
        const int ca = pa - rect.a0, cb = c.bbase + rb - rect.b0;
        if (!sf_any(mine && (ta > xs + 4.5f || tb > ys + 3.5f))) {
            patch(xs, ca, ys, cb);  // nearly always
        } else {
            for (int h = 0; h < kSfQuads && sf_any(mine && ta > xs + (float)(4 * h) + 0.5f); ++h)
                for (int e = 0; e < kSfQuads && sf_any(mine && tb > ys + (float)(3 * e) + 0.5f); ++e)
                    patch(xs + (float)(4 * h), ca + 4 * h, ys + (float)(3 * e), cb + 3 * e);
        }
        if (sf_any(m != 0.0f && !fits)) {
            if (m != 0.0f && !fits) {
                SfFootprint f;
                sf_unbox<KIND>(x, c, s, f);
                sf_for_each<KIND>(f, [&](int a, int b, float w) {
                    atomicAdd(img + (unsigned)(b * s.nu + a), w * scale);
                });
            }
        }
    }
}

template <int KIND>
__global__ __launch_bounds__(kSfBx * kSfBy, 4) void sf_fwd_kernel(GeoScalars s, int steps,
                                                                  const ViewGeo* __restrict__ views,
                                                                  const float* __restrict__ vol,
                                                                  float* __restrict__ proj)
{
    // per wavefront a tile, then a dump for the four columns of a row outside it
    // (of static size it costs four to five more spilled registers)
    extern __shared__ float tiles[];
    const ViewGeo& g = views[blockIdx.y];
    float* img = proj + (size_t)blockIdx.y * s.nu * s.nv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.y), lane = threadIdx.x;
    float* tile = tiles + wave * (kSfTile + kSfPatchCols);
    double src[3];
    const int dom = __builtin_amdgcn_readfirstlane(sf_source(g, s, src));
    // across: the lanes' axis, along: the other one
    const int across = dom == 0 ? s.ny : s.nx, along = dom == 0 ? s.nx : s.ny;
    const int nta = (across + kSfBx - 1) / kSfBx;
    const int brick = blockIdx.x * kSfBy + wave;
    const int p0 = (brick % nta) * kSfBx, q0 = (brick / nta) * steps;
    if (q0 >= along) return;  // (wavefronts are independent: no barriers)
    const int p1 = min(p0 + kSfBx, across) - 1, q1 = min(q0 + steps, along) - 1;
    const int kb = blockIdx.z * kSfCol, nk = min(kSfCol, s.nz - kb);
    const size_t plane = (size_t)s.nx * s.ny;
    const bool active = p0 + lane <= p1;
    const int p = min(p0 + lane, p1);
    // as many voxels along z at once as the tile has room for
    int sub = nk;
    for (int k0 = 0; k0 < nk; k0 += sub) {
        SfRect rect;
        for (;; sub = (sub + 1) / 2) {
            const int ka = kb + k0, ke = min(ka + sub, kb + nk) - 1;
            rect = dom == 0 ? sf_rect(g, s, q0, q1, p0, p1, ka, ke) : sf_rect(g, s, p0, p1, q0, q1, ka, ke);
            if (!rect.known || rect.w * rect.h <= kSfTile || sub == 1) break;
        }
        const int ke = min(sub, nk - k0);
        const int npix = rect.w * rect.h;
        if (rect.known && npix == 0) continue;  // no footprint of these voxels reaches the detector
        const bool tiled = rect.known && npix <= kSfTile && s.nu >= 4;
        if (tiled)
            for (int t = lane; t < npix; t += 64) tile[t] = 0.0f;
        for (int q = q0; q <= q1; ++q) {
            const int i = dom == 0 ? q : p, j = dom == 0 ? p : q;
            const float* mu = vol + (size_t)(kb + k0) * plane + (size_t)j * s.nx + i;
            bool any = false;
            for (int kk = 0; kk < ke; ++kk) any = any || mu[kk * plane] != 0.0f;
            if (!sf_any(active && any)) continue;
            const SfColumn col = sf_column<KIND>(g, s, src, dom, i, j, kb + kSfCol / 2);
            if (tiled && !sf_any(!col.front)) {
                sf_scatter<KIND>(col, s, dom, kb + k0, ke, mu, plane, active, rect, tile, img);
                continue;
            }
            if (active)
                for (int kk = 0; kk < ke; ++kk) {
                    const float m = mu[kk * plane];
                    SfFootprint f;
                    if (m == 0.0f || !sf_voxel<KIND>(col, g, s, src, dom, i, j, kb + k0 + kk, f)) continue;
                    const float scale = f.L * m;
                    sf_for_each<KIND>(f, [&](int a, int b, float w) {
                        atomicAdd(img + (unsigned)(b * s.nu + a), w * scale);
                    });
                }
        }
        if (tiled) {
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            for (int t = lane; t < npix; t += 64) {
                const float v = tile[t];
                const int b = t / rect.w, a = t - b * rect.w;
                if (v != 0.0f) atomicAdd(img + (unsigned)((rect.b0 + b) * s.nu + rect.a0 + a), v);
            }
        }
    }
}

// Back-projection: a thread owns kSfCol voxels along z, whose FP64 sums over
// the views stay in LDS.
template <int KIND>
__global__ __launch_bounds__(kSfBx * kSfBy, 4) void sf_bp_kernel(GeoScalars s, int V,
                                                              const ViewGeo* __restrict__ views,
                                                              const float* __restrict__ proj,
                                                              float* __restrict__ vol)
{
    __shared__ double sum[kSfCol][kSfBx * kSfBy];
    const int i = blockIdx.x * kSfBx + threadIdx.x;
    const int j = blockIdx.y * kSfBy + threadIdx.y;
    const int kb = blockIdx.z * kSfCol, nk = min(kSfCol, s.nz - kb);
    const int tid = threadIdx.y * kSfBx + threadIdx.x;
    if (i >= s.nx || j >= s.ny) return;
    for (int kk = 0; kk < kSfCol; ++kk) sum[kk][tid] = 0.0;
    for (int v = 0; v < V; ++v) {
        const ViewGeo& g = views[v];
        double src[3];
        const int dom = sf_source(g, s, src);
        const SfImage img{proj + (size_t)v * s.nu * s.nv, s.nu};
        const SfColumn col = sf_column<KIND>(g, s, src, dom, i, j, kb + kSfCol / 2);
        sf_walk<KIND>(col, g, s, src, dom, i, j, kb, nk, img, [](int) { return true; },
                      [&](int kk, int, const float (&acc)[1]) { sum[kk][tid] += acc[0]; });
    }
    for (int kk = 0; kk < nk; ++kk) vol[((size_t)(kb + kk) * s.ny + j) * s.nx + i] = (float)sum[kk][tid];
}

// Per-view block reduction of C channels into partials[v][blk][C] (fixed
// order: wavefront butterflies, then the 4 wavefronts in sequence).  At the
// first butterfly steps each lane keeps half of its channels and receives the
// partner's sums of them, so C channels take about C + log C exchanges
// instead of 6 C; the additions are those of the full butterfly.
template <int N>
__device__ inline void sf_halve(float (&r)[N], float (&o)[(N + 1) / 2], bool high, int off)
{
    constexpr int H = (N + 1) / 2;
#pragma unroll
    for (int t = 0; t < H; ++t) {
        const float up = H + t < N ? r[H + t] : 0.0f;
        const float keep = high ? up : r[t], give = high ? r[t] : up;
        o[t] = keep + __shfl_xor(give, off);
    }
}

// The steps after the first: r1 holds the half of the C channels that the
// lane kept (the first (C + 1) / 2 in lanes 0 .. 31).
template <int C>
__device__ inline void sf_reduce_half(float (&r1)[(C + 1) / 2], float (&red)[kSfBy][C], float* out)
{
    constexpr int C1 = (C + 1) / 2, C2 = (C1 + 1) / 2;
    const int lane = threadIdx.x, wave = threadIdx.y;
    float r2[C2];
    sf_halve(r1, r2, (lane & 16) != 0, 16);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1)
#pragma unroll
        for (int t = 0; t < C2; ++t) r2[t] += __shfl_xor(r2[t], off);
    if ((lane & 15) == 0) {
        // lanes 0, 16, 32, 48 hold the channels from 0, C2, C1, C1 + C2 on
        const int first = (lane & 32 ? C1 : 0) + (lane & 16 ? C2 : 0);
        const int last = min(lane & 32 ? C : C1, (lane & 16) ? first + C1 : first + C2);
#pragma unroll
        for (int t = 0; t < C2; ++t)
            if (first + t < last) red[wave][first + t] = r2[t];
    }
    __syncthreads();
    if (wave == 0 && lane < C) out[lane] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    __syncthreads();
}

__device__ inline float vol_at(const float* __restrict__ v, const GeoScalars& s, int i, int j, int k)
{
    if (i < 0 || j < 0 || k < 0 || i >= s.nx || j >= s.ny || k >= s.nz) return 0.0f;
    return v[((size_t)k * s.ny + j) * s.nx + i];
}

// The pose-gradient kernels: `split` blocks share a brick's views (a small
// volume alone would leave CUs idle); the partial sums are per view and block,
// the same whatever the split.
template <int KIND>
__global__ __launch_bounds__(kSfBx * kSfBy, 4) void sf_fwd_grad_kernel(GeoScalars s, int V, int split,
                                                                    const ViewGeo* __restrict__ views,
                                                                    const float* __restrict__ vol,
                                                                    const float* __restrict__ grad_proj,
                                                                    float* __restrict__ partials)
{
    __shared__ float red[kSfBy][kRdChannels];
    __shared__ float G[kSfCol][3][kSfBx * kSfBy];
    const int i = blockIdx.x * kSfBx + threadIdx.x;
    const int j = blockIdx.y * kSfBy + threadIdx.y;
    const int bz = blockIdx.z / split, vstart = blockIdx.z % split;
    const int kb = bz * kSfCol, nk = min(kSfCol, s.nz - kb);
    const int blk = (bz * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int nblk = gridDim.x * gridDim.y * (gridDim.z / split);
    const int tid = threadIdx.y * kSfBx + threadIdx.x;
    // central-difference gradient (index units: half the neighbour difference)
    bool any = false;
    if (i < s.nx && j < s.ny)
        for (int kk = 0; kk < nk; ++kk) {
            const int k = kb + kk;
            const float gx = 0.5f * (vol_at(vol, s, i + 1, j, k) - vol_at(vol, s, i - 1, j, k));
            const float gy = 0.5f * (vol_at(vol, s, i, j + 1, k) - vol_at(vol, s, i, j - 1, k));
            const float gz = 0.5f * (vol_at(vol, s, i, j, k + 1) - vol_at(vol, s, i, j, k - 1));
            G[kk][0][tid] = gx;
            G[kk][1][tid] = gy;
            G[kk][2][tid] = gz;
            any = any || !(gx == 0.0f && gy == 0.0f && gz == 0.0f);
        }
    const float pi = (float)i - 0.5f * (s.nx - 1), pj = (float)j - 0.5f * (s.ny - 1);
    for (int v = vstart; v < V; v += split) {
        const ViewGeo& g = views[v];
        float r[kRdChannels];
#pragma unroll
        for (int ch = 0; ch < kRdChannels; ++ch) r[ch] = 0.0f;
        if (any) {  // columns of a uniform region need no projection
            double src[3];
            const int dom = sf_source(g, s, src);
            const SfImage w{grad_proj + (size_t)v * s.nu * s.nv, s.nu};
            const SfColumn col = sf_column<KIND>(g, s, src, dom, i, j, kb + kSfCol / 2);
            sf_walk<KIND>(
                col, g, s, src, dom, i, j, kb, nk, w,
                [&](int kk) {
                    return !(G[kk][0][tid] == 0.0f && G[kk][1][tid] == 0.0f && G[kk][2][tid] == 0.0f);
                },
                [&](int kk, int k, const float (&sj)[1]) {
                    const float pk = (float)k - 0.5f * (s.nz - 1);
                    const float gx = sj[0] * G[kk][0][tid], gy = sj[0] * G[kk][1][tid],
                                gz = sj[0] * G[kk][2][tid];
                    // B_c, then T_xy, T_xz, T_yx, T_yz, T_zx, T_zy (T_ac = sum s P_a G_c)
                    r[0] += gx; r[1] += gy; r[2] += gz;
                    r[3] = fmaf(pi, gy, r[3]); r[4] = fmaf(pi, gz, r[4]);
                    r[5] = fmaf(pj, gx, r[5]); r[6] = fmaf(pj, gz, r[6]);
                    r[7] = fmaf(pk, gx, r[7]); r[8] = fmaf(pk, gy, r[8]);
                });
        }
        float r1[(kRdChannels + 1) / 2];
        sf_halve(r, r1, (threadIdx.x & 32) != 0, 32);
        sf_reduce_half<kRdChannels>(r1, red, partials + ((size_t)v * nblk + blk) * kRdChannels);
    }
}

// Views [v0, v0 + Vc) (split as above); grad_img holds this chunk's detector gradient images.
template <int KIND>
__global__ __launch_bounds__(kSfBx * kSfBy, 4) void sf_bp_grad_kernel(GeoScalars s, int v0, int Vc, int split,
                                                                   const ViewGeo* __restrict__ views,
                                                                   const float2* __restrict__ grad_img,
                                                                   const float* __restrict__ grad_vol,
                                                                   float* __restrict__ partials)
{
    __shared__ float red[kSfBy][kVdChannels];
    __shared__ float E[kSfCol][kSfBx * kSfBy];
    const int i = blockIdx.x * kSfBx + threadIdx.x;
    const int j = blockIdx.y * kSfBy + threadIdx.y;
    const int bz = blockIdx.z / split, vstart = blockIdx.z % split;
    const int kb = bz * kSfCol, nk = min(kSfCol, s.nz - kb);
    const int blk = (bz * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int nblk = gridDim.x * gridDim.y * (gridDim.z / split);
    const int tid = threadIdx.y * kSfBx + threadIdx.x;
    bool any = false;
    if (i < s.nx && j < s.ny)
        for (int kk = 0; kk < nk; ++kk) {
            const float e = grad_vol[((size_t)(kb + kk) * s.ny + j) * s.nx + i];
            E[kk][tid] = e;
            any = any || e != 0.0f;
        }
    const float pi = (float)i - 0.5f * (s.nx - 1), pj = (float)j - 0.5f * (s.ny - 1);
    for (int vv = vstart; vv < Vc; vv += split) {
        const int v = v0 + vv;
        const ViewGeo& g = views[v];
        float A1 = 0.f, A2 = 0.f, A3 = 0.f, Z1 = 0.f, Z2 = 0.f, Z3 = 0.f;
        if (any) {
            double src[3];
            const int dom = sf_source(g, s, src);
            const SfGradImage img{grad_img + (size_t)vv * s.nu * s.nv, s.nu};
            const SfColumn col = sf_column<KIND>(g, s, src, dom, i, j, kb + kSfCol / 2);
            sf_walk<KIND>(
                col, g, s, src, dom, i, j, kb, nk, img, [&](int kk) { return E[kk][tid] != 0.0f; },
                [&](int kk, int k, const float (&d)[2]) {
                    const float da = d[0], db = d[1];
                    // projection of the voxel centre: offsets from the detector centre (pixels), depth
                    float ap, bp, Wc;
                    if (col.fast) {
                        const float dk = (float)k - col.ka;
                        Wc = fmaf(dk, col.pwz, col.bw);
                        const float iw = __builtin_amdgcn_rcpf(Wc);
                        ap = col.uco + fmaf(dk * col.ucn, iw, col.ucfr);
                        bp = col.bco + fmaf(dk * col.bn, iw, col.bfr);
                    } else {
                        const double fi = i, fj = j, fk = k;
                        const double U = fma(g.PUd[0], fi, fma(g.PUd[1], fj, fma(g.PUd[2], fk, g.PUd[3])));
                        const double Vv = fma(g.PVd[0], fi, fma(g.PVd[1], fj, fma(g.PVd[2], fk, g.PVd[3])));
                        const double W = fma(g.PWd[0], fi, fma(g.PWd[1], fj, fma(g.PWd[2], fk, g.PWd[3])));
                        Wc = (float)W;
                        ap = (float)(U / W);
                        bp = (float)(Vv / W);
                    }
                    const float ec = E[kk][tid] * __builtin_amdgcn_rcpf(Wc);
                    const float c1 = ec * da, c2 = ec * db;
                    const float c3 = -ec * fmaf(da, ap, db * bp);
                    const float pk = (float)k - 0.5f * (s.nz - 1);
                    A1 += c1; A2 += c2; A3 += c3;
                    Z1 = fmaf(c1, pk, Z1); Z2 = fmaf(c2, pk, Z2); Z3 = fmaf(c3, pk, Z3);
                });
        }
        // channels A, pi A, pj A, Z: lanes 0 .. 31 keep the first six.  A
        // lower lane's product with its (pi, pj) is added unrounded.
        const bool high = (threadIdx.x & 32) != 0;
        const float A[3] = {A1, A2, A3}, Z[3] = {Z1, Z2, Z3};
        float r1[kVdChannels / 2];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const float ra = __shfl_xor(A[t], 32), rb = __shfl_xor(high ? pi * A[t] : Z[t], 32);
            r1[t] = high ? fmaf(pj, ra, pj * A[t]) : A[t] + ra;
            r1[3 + t] = high ? Z[t] + rb : fmaf(pi, A[t], rb);
        }
        sf_reduce_half<kVdChannels>(r1, red, partials + ((size_t)v * nblk + blk) * kVdChannels);
    }
}

__global__ void sf_zero_kernel(size_t n, float* __restrict__ p)
{
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        p[t] = 0.0f;
}

static dim3 sf_grid(const GeoScalars& s, int split = 1)
{
    return dim3((s.nx + kSfBx - 1) / kSfBx, (s.ny + kSfBy - 1) / kSfBy, (s.nz + kSfCol - 1) / kSfCol * split);
}

int sf_blocks(const GeoScalars& s)
{
    const dim3 g = sf_grid(s);
    return (int)(g.x * g.y * g.z);
}

// How many blocks share the V views of a brick: enough for about 2048 blocks (64^3,
// 8 views, SF forward and gradient 150 -> 105 us).
static int sf_view_split(const GeoScalars& s, int V)
{
    return std::max(1, std::min(V, 2048 / sf_blocks(s)));
}

#define DP_FP_LAUNCH(KERNEL, SPLIT, ...)                                                           \
    do {                                                                                    \
        if (kind == kFpDD)                                                                  \
            KERNEL<kFpDD><<<sf_grid(s, SPLIT), dim3(kSfBx, kSfBy), 0, st>>>(__VA_ARGS__);          \
        else                                                                                \
            KERNEL<kFpSF><<<sf_grid(s, SPLIT), dim3(kSfBx, kSfBy), 0, st>>>(__VA_ARGS__);          \
    } while (0)

void launch_sf_fwd(const GeoScalars& s, int V, const ViewGeo* views, const float* vol, float* proj,
                   int kind, hipStream_t st)
{
    const size_t n = (size_t)V * s.nu * s.nv;
    const int fill = (int)std::min<size_t>((n + 255) / 256, 65536);
    // Enough bricks (one per wavefront, in either lane order: each view picks
    // its own) to fill the chip; beyond that, bricks deeper along the rays,
    // whose pixels take more voxels each before they go to memory.
    const auto bricks = [&](int steps) {
        return std::max(((s.nx + kSfBx - 1) / kSfBx) * ((s.ny + steps - 1) / steps),
                        ((s.ny + kSfBx - 1) / kSfBx) * ((s.nx + steps - 1) / steps));
    };
    const int zb = (s.nz + kSfCol - 1) / kSfCol;
    int steps = kSfSteps;
    while (steps > 1 && (long long)bricks(steps) * V * zb < kSfFwdWaves) steps /= 2;
    const dim3 grid((bricks(steps) + kSfBy - 1) / kSfBy, V, zb), block(kSfBx, kSfBy);
    constexpr size_t lds = kSfBy * (kSfTile + kSfPatchCols) * sizeof(float);
    prof_begin(DP_K_SF, st);
    sf_zero_kernel<<<fill, 256, 0, st>>>(n, proj);
    if (kind == kFpDD) sf_fwd_kernel<kFpDD><<<grid, block, lds, st>>>(s, steps, views, vol, proj);
    else sf_fwd_kernel<kFpSF><<<grid, block, lds, st>>>(s, steps, views, vol, proj);
    prof_end(DP_K_SF, st);
}

void launch_sf_bp(const GeoScalars& s, int V, const ViewGeo* views, const float* proj, float* vol,
                  int kind, hipStream_t st)
{
    prof_begin(DP_K_SF, st);
    DP_FP_LAUNCH(sf_bp_kernel, 1, s, V, views, proj, vol);
    prof_end(DP_K_SF, st);
}

void launch_sf_fwd_grad(const GeoScalars& s, int V, const ViewGeo* views, const float* vol,
                        const float* grad_proj, float* partials, int kind, hipStream_t st)
{
    prof_begin(DP_K_SF, st);
    const int split = sf_view_split(s, V);
    DP_FP_LAUNCH(sf_fwd_grad_kernel, split, s, V, split, views, vol, grad_proj, partials);
    prof_end(DP_K_SF, st);
}

void launch_sf_bp_grad(const GeoScalars& s, int v0, int Vc, const ViewGeo* views,
                       const float2* grad_img, const float* grad_vol, float* partials, int kind,
                       hipStream_t st)
{
    prof_begin(DP_K_SF, st);
    const int split = sf_view_split(s, Vc);
    DP_FP_LAUNCH(sf_bp_grad_kernel, split, s, v0, Vc, split, views, grad_img, grad_vol, partials);
    prof_end(DP_K_SF, st);
}
#undef DP_FP_LAUNCH

}  // namespace dp
