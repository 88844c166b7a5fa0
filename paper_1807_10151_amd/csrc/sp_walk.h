// Index arithmetic of the projector pair, shared by the kernels and the host
// index checker (all __host__ __device__): the ray a lane of R owns, the
// major-step range and the padded minor coordinate of its walk, and the first
// candidate bin of a pixel in R^T.  Coordinates are in pixel units with the
// image centred at the origin (pixel centre x_j = j - xoff, y_i = yoff - i).
#pragma once

#include "sp_internal.h"

namespace sp {

// Ray of lane `lane` of wave W: index ai of the class-sorted angle table and
// bin k; false for a lane past the end of its class, its tail stream or the
// bins.
__host__ __device__ inline bool wave_ray(const WaveDev& W, int lane, int nB, int& ai, int& k) {
    if (W.tail == WAVE_BLOCK) {
        ai = W.a0 + lane / WAVE_BINS;
        k = W.k0 + lane % WAVE_BINS;
        return ai < W.aend && k < nB;
    }
    if (W.tail == WAVE_ROW) {
        ai = W.a0;
        k = W.k0 + lane;
        return k < nB;
    }
    const int r = nB % WAVE_BINS;
    const int e = W.k0 + lane;
    ai = W.a0 + e / r;
    k = nB - r + e % r;
    return ai < W.aend;
}

// First ray (ai, k) of lane `lane`'s pair (k, k + 1) in wave W of the two-ray
// form's oblique kinds; the second ray exists when k + 1 < nB.
__host__ __device__ inline bool wave_pair(const WaveDev& W, int lane, int nB, int& ai, int& k) {
    int q;
    const bool ok = wave_ray(WaveDev{W.a0, W.k0, W.aend, W.tail - WAVE_PAIR_BLOCK}, lane, (nB + 1) / 2, ai, q);
    k = 2 * q;
    return ok;
}

// Fractional minor index where ray (A, sk) crosses the centre line of major
// step 0 (row 0 for vertical angles, column 0 for horizontal ones), minus the
// half-width hw of its nonzero band: the axis walk's candidate reference.
template <bool HORIZ>
__host__ __device__ inline double walk_start(const GeomDev& G, const AngleDev& A, double sk) {
    return (HORIZ ? G.yoff - (sk + G.xoff * A.c) / A.s : (sk - G.yoff * A.s) / A.c + G.xoff) -
           (double)A.hw;
}

// Padded minor coordinate (pixel q spans [q, q + 1) after the PAD offset)
// where an oblique ray enters major band 0 on its lower side: band m is then
// met over [b0 + m slope, b0 + m slope + |slope|].
template <bool HORIZ>
__host__ __device__ inline double split_b0(const GeomDev& G, const AngleDev& A, double sk) {
    return (HORIZ ? G.yoff + 0.5 - (sk + (G.xoff + 0.5) * A.c) / A.s
                  : (sk - (G.yoff + 0.5) * A.s) / A.c + G.xoff + 0.5) +
           fmin(A.slope, 0.0) + (double)PAD;
}

// Major-axis steps [lo, hi) of [0, n) where base + m * slope lies in [vlo, vhi],
// widened by one step on each side (a superset of the steps where the ray
// meets the image).
__host__ __device__ inline void step_range(double base, double slope, double vlo, double vhi,
                                           int n, int& lo, int& hi) {
    if (slope == 0.0) {
        const bool in = base >= vlo && base <= vhi;
        lo = 0;
        hi = in ? n : 0;
        return;
    }
    const double t0 = (vlo - base) / slope, t1 = (vhi - base) / slope;
    double tmin = fmin(t0, t1) - 1.0, tmax = fmax(t0, t1) + 2.0;
    tmin = fmin(fmax(tmin, 0.0), (double)n);
    tmax = fmin(fmax(tmax, 0.0), (double)n);
    lo = (int)floor(tmin);
    hi = (int)ceil(tmax);
    if (hi < lo) hi = lo;
}

// One lane's step range of its ray (before the wave's union is taken).
template <bool HORIZ>
__host__ __device__ inline void ray_steps(const GeomDev& G, const AngleDev& A, double sk, int& lo,
                                          int& hi) {
    const int nmaj = HORIZ ? G.cols : G.rows;
    const int nmin = HORIZ ? G.rows : G.cols;
    step_range(walk_start<HORIZ>(G, A, sk), A.slope, -(double)(A.nc + 1), (double)(nmin + 1), nmaj,
               lo, hi);
}

// The two-ray form.  pair_swap: the pair's ray of bin k has the larger padded
// minor coordinate.  The lower ray walks as ray_split's; the upper one is
// `delta` further, 1 <= delta < 2, so with j the lower ray's first pixel the
// two meet at most pixels j .. j + 1 and j + 1 .. j + 3.
template <bool HORIZ>
__host__ __device__ inline bool pair_swap(const AngleDev& A) {
    return HORIZ ? A.s > 0.0 : A.c < 0.0;
}
__host__ __device__ inline double pair_delta(const GeomDev& G, const AngleDev& A) { return G.ds * A.wmax; }
__host__ __device__ inline bool pair_fits(const GeomDev& G, const AngleDev& A) {
    const double d = pair_delta(G, A);
    return G.ds >= 1.0 && d >= 1.0 && d < 2.0 - 1e-6;
}
// Shares of a band's path length, from the fraction fr of the lower ray's
// padded minor coordinate and isg = 1 / |slope|: f, of the lower ray in pixel
// j (the rest in j + 1); g1, of the upper ray in pixels up to j + 1, and g2, up
// to j + 2 (the rest in j + 3).
__host__ __device__ inline void pair_shares(double fr, double isg, double delta, double& f, double& g1,
                                            double& g2) {
    f = fmin(fmax(fma(fr, -isg, isg), 0.0), 1.0);
    g1 = fmin(fmax(fma(fr, -isg, (2.0 - delta) * isg), 0.0), 1.0);
    g2 = fmin(fmax(fma(fr, -isg, (3.0 - delta) * isg), 0.0), 1.0);
}

// Steps [lo, hi) of part `part` of nparts of a wave's common range [lo, hi).
__host__ __device__ inline void part_range(int& lo, int& hi, int part, int nparts) {
    if (nparts > 1 && hi > lo) {
        const int len = hi - lo;
        const int l0 = lo + len * part / nparts;
        hi = lo + len * (part + 1) / nparts;
        lo = l0;
    }
}

// R^T: window index kf = t / ds + kb of a pixel whose centre (xj, yi)
// projects to t = xj c + yi s on the angle's normal.  The pixel's candidate
// bins are the NB bins from padded index trunc(kf) (bin trunc(kf) - PAD).
// Axis-parallel angles form t exactly and divide; oblique ones fold 1/ds into
// the angle's constants (kc = yi s / ds + kb is shared by a lane's pixels),
// and their first candidate's offset s_k - t is dc - ds fract(kf).
__host__ __device__ inline double bp_kf(double t, double inv_ds, double kb) {
    return fma(t, inv_ds, kb);
}
__host__ __device__ inline double bp_kc(double yi, const AngleDev& A) { return fma(yi, A.sids, A.kb); }
__host__ __device__ inline double bp_kf_oblique(double xj, double kc, const AngleDev& A) {
    return fma(xj, A.cids, kc);
}

// R^T over 2 x 2 blocks (see BpAngle): the window index of the block with
// centre (xc, yc), the scaled offset w of the window's first bin from pixel
// A's centre, and the weights of each pixel's bins in the three-bin window.
__host__ __device__ inline double bp_quad_kf(double xc, double yc, const BpAngle& Q) {
    return fma(xc, Q.cids, fma(yc, Q.sids, Q.kb));
}
__host__ __device__ inline double bp_quad_w(double fract_kf, const BpAngle& Q) {
    return fma(fract_kf, Q.nk, Q.wc);
}
__host__ __device__ inline double clamp01(double v) { return fmin(fmax(v, 0.0), 1.0); }
__host__ __device__ inline void bp_quad_a(const BpAngle& Q, double w, double (&u)[2]) {   // bins 0, 1
    u[0] = clamp01(Q.einv - fabs(w));
    u[1] = clamp01(Q.eK - w);
}
__host__ __device__ inline void bp_quad_b(const BpAngle& Q, double w, double (&u)[3]) {
    u[0] = clamp01(Q.einv - fabs(w + Q.dB0));
    u[1] = clamp01(Q.einv - fabs(w + Q.dB1));
    u[2] = clamp01(Q.eB2 - w);
}
__host__ __device__ inline void bp_quad_c(const BpAngle& Q, double w, double (&u)[3]) {
    u[0] = clamp01(Q.eC0 + w);
    u[1] = clamp01(Q.einv - fabs(w + Q.dC1));
    u[2] = clamp01(Q.eC2 - w);
}
__host__ __device__ inline void bp_quad_d(const BpAngle& Q, double w, double (&u)[2]) {   // bins 1, 2
    u[0] = clamp01(Q.einv - fabs(w + Q.dD1));
    u[1] = clamp01(Q.einv - fabs(w + Q.dD2));
}
// Corner (A 0, B 1, C 2, D 3) of the block's pixel p = 2 r + c (row r, column c).
__host__ __device__ inline int bp_quad_corner(int run, int p) {
    const int n = p ^ (run & (BP_FLIP_X | BP_FLIP_Y));   // bit 0: towards larger t along x, bit 1: along y
    const bool vert = run & BP_VERT;                     // |c| >= |s|: B is the neighbour along y
    return n == 0 || n == 3 ? n : ((n == 2) == vert ? 1 : 2);
}

// Tile (bx, by) of R^T's gx x gy tile grid that launch-order workgroup `id`
// takes.  Workgroups go to the 8 XCDs round-robin in launch order (id mod 8);
// when the grid splits into 4 x 2 equal regions, XCD q takes region
// (q mod 4, q / 4), row by row: a compact image region projects onto a narrow
// band of each sinogram row, so each XCD's L2 holds fewer windows.  Otherwise
// row-major.  The tiles' sums do not depend on the order.
__host__ __device__ inline void bp_tile_of(int id, int gx, int gy, int& bx, int& by) {
    if ((gx & 3) == 0 && (gy & 1) == 0) {
        const int q = id & 7, jj = id >> 3, rw = gx >> 2, rh = gy >> 1;
        bx = (q & 3) * rw + jj % rw;
        by = (q >> 2) * rh + jj / rw;
    } else {
        bx = id % gx;
        by = id / gx;
    }
}

}  // namespace sp
