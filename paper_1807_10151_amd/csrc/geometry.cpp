// Host side of the geometry: the class-sorted angle table (Section 4.1's
// equally spaced angles, cos/sin snapped at multiples of pi/4), the bin
// positions, R's wave table and dispatch order, and the launch shapes of R and
// R^T.  Plain C++ with no runtime calls, so that the index checker can build it
// on the host alone.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <vector>

#include "../../include/suppcg.h"
#include "sp_internal.h"
#include "sp_walk.h"

namespace sp {

void angle_cos_sin(const sp_geometry& g, int a, double& co, double& si) {
    const double dth = g.dtheta > 0.0 ? g.dtheta : M_PI / g.n_angles;
    const double th = g.theta0 + a * dth;
    const double q = th / (M_PI / 4.0);
    const double m = std::nearbyint(q);
    if (std::fabs(q - m) < 1e-12) {
        static const double h = std::sqrt(0.5);
        static const double tc[8] = {1.0, h, 0.0, -h, -1.0, -h, 0.0, h};
        static const double ts[8] = {0.0, h, 1.0, h, 0.0, -h, -1.0, -h};
        long long mi = (long long)m % 8;
        if (mi < 0) mi += 8;
        co = tc[mi];
        si = ts[mi];
    } else {
        co = std::cos(th);
        si = std::sin(th);
    }
}

AngleDev angle_entry(const sp_geometry& g, int a, double ds, double s0, double margin) {
    double co, si;
    angle_cos_sin(g, a, co, si);
    AngleDev A{};
    A.c = co;
    A.s = si;
    const double ac = std::fabs(co), as = std::fabs(si);
    const bool axis = ac == 0.0 || as == 0.0;
    const bool horiz = as > ac;
    const double e = 0.5 * (ac + as);
    const double inv = axis ? 0.0 : 1.0 / std::min(ac, as);
    A.inv = inv;
    A.einv = e * inv;
    A.wmax = 1.0 / std::max(ac, as);
    A.slope = horiz ? co / si : si / co;
    const double hw = e / std::max(ac, as) + margin;
    A.hw = (float)hw;
    A.nc = (int)std::ceil(2.0 * hw);
    const double hb = (e + margin) / ds;
    A.nb = (int)std::ceil(2.0 * hb);
    A.kb = -s0 / ds - hb + 1.0 + PAD;
    A.dc = ds * (1.0 - hb);
    A.cids = co / ds;
    A.sids = si / ds;
    A.row = a;
    A.flags = (axis ? ANG_AXIS : 0) | (horiz ? ANG_HORIZ : 0);
    return A;
}

int angle_class(const AngleDev& A) {
    const bool axis = A.flags & ANG_AXIS, horiz = A.flags & ANG_HORIZ;
    return (axis ? 2 : 0) + (horiz ? 1 : 0);
}

namespace {
int geom_fail(char* err, size_t n, const char* fmt, ...) {
    if (err && n) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(err, n, fmt, ap);
        va_end(ap);
    }
    return SP_ERR_ARG;
}
}  // namespace

namespace {
// The wave table of R's one-ray form, or of its two-ray form over pairs of bins.
int wave_table(const GeomDev& G, bool pair, WaveDev* out) {
    // Oblique classes: waves of WAVE_ANGLES angles by WAVE_BINS bins, a
    // workgroup's four waves the four 16-bin sub-chunks of one 64-bin chunk
    // for the same four neighbouring angles (rays that cross nearly the same
    // pixels), chunk by chunk; then the classes' packed tails (the last
    // nB % WAVE_BINS bins).  Axis-parallel classes: waves of 64 bins of one
    // angle.  The dispatch order sorts workgroups by cost and keeps this
    // order among equal costs, so workgroups that run side by side on the GPU
    // read neighbouring parts of the image.
    const int nB = pair ? (G.nB + 1) / 2 : G.nB, kind = pair ? WAVE_PAIR_BLOCK : WAVE_BLOCK;
    const int r = nB % WAVE_BINS, full = nB / WAVE_BINS;
    int w = 0;
    auto put = [&](const WaveDev& W) {
        if (out) out[w] = W;
        ++w;
    };
    for (int c = 0; c < full; c += 4)
        for (int q = 0; q < 2; ++q) {
            const int a0 = G.cls[q], a1 = G.cls[q + 1];
            for (int g0 = a0; g0 < a1; g0 += WAVE_ANGLES)
                for (int j = c; j < std::min(full, c + 4); ++j) put(WaveDev{g0, WAVE_BINS * j, a1, kind});
        }
    for (int q = 0; q < 2; ++q) {
        const int a0 = G.cls[q], a1 = G.cls[q + 1];
        if (r == 0) continue;
        const int stream = (a1 - a0) * r;
        for (int e = 0; e < stream; e += 64) put(WaveDev{a0, e, a1, kind + (WAVE_TAIL - WAVE_BLOCK)});
    }
    for (int q = 2; q < 4; ++q)
        for (int a = G.cls[q]; a < G.cls[q + 1]; ++a)
            for (int k0 = 0; k0 < G.nB; k0 += 64) put(WaveDev{a, k0, a + 1, WAVE_ROW});
    return w;
}
}  // namespace

int project_wave_count(const GeomDev& G) { return project_waves(G, nullptr); }
int project_waves(const GeomDev& G, WaveDev* out) { return wave_table(G, false, out); }
int project_pair_waves(const GeomDev& G, WaveDev* out) { return wave_table(G, true, out); }

void project_shape(GeomDev& G, int resident_waves) {
    const long W = resident_waves, nw = G.nwaves, side = ((long)G.rows + G.cols) / 2;
    const bool longest = std::max(G.rows, G.cols) > 512;
    auto set = [&](long parts, bool mem) {
        G.parts = (int)parts;
        G.pmem = mem ? 1 : 0;
    };
    // Large images: 8 parts keep the resident waves on a band of the float64
    // copies (measured: 2048^2 x 2048 angles 9.3 -> 5.8 ms).
    if ((long)G.rows * G.cols >= (1L << 21)) return set(8, true);
    // Otherwise split only a grid that would leave wave slots empty.  Parts summed
    // in one workgroup save the second launch and the traffic of the sums, but a
    // workgroup of 8 or 16 waves needs a CU's slots in one piece: a grid that
    // exceeds a round of them (4 parts: a quarter of W waves, 2: a half) takes two
    // (the last and shortest workgroups apart).  Times of one call in us:
    if (10 * nw >= 9 * W) return set(1, false);
    if (side > 512) {
        // Long walks: any such tail costs more than the launch.  8 parts where 4 (or
        // 3, 2) fill the slots; 900^2 x 150 angles, 3 parts in the workgroup /
        // through memory / 8 through memory 106 / 75 / 76, 1300^2 x 36 (4 parts) 80
        // / 77 / 63; 600^2 x 320 (2 parts) 70 / 75 / 75.
        if (side < 724 && 2 * nw > W && 8 * nw <= 5 * W) return set(2, false);
        return set(8, true);
    }
    // Short walks: one workgroup's 13 - 25 against 17 - 30; 100^2 x 1000 angles, 4 /
    // 2 / 1 parts 20 / 17 / 21, x 2000 26 / 24 / 22.
    if (side <= 128) return set(4 * nw <= W ? 4 : (2 * nw <= W ? 2 : 1), false);
    // Few angles for the image's size (1.4 per pixel of a side are 0.03 waves per
    // square pixel), or a grid between the two rounds: through memory, but where
    // the workgroups are about one per CU.  400^2 x 180 angles, 4 parts 36 / 33, x
    // 230 (3 parts) 51 / 40, x 113 30 / 31; 300^2 x 390 (3) 42 / 32.
    const bool few = 54 * nw < side * side || (longest && 2 * nw < W);
    const bool between = side >= 280 && 3 * nw > W && 5 * nw < 2 * W;
    if ((few && 32 * nw > 5 * W) || between) return set(std::min(4L, (W + nw - 1) / nw), true);
    // 243^2 x 360, 4 parts 24 / 27; 340^2 x 476, 2 in the workgroup / 3 through memory
    // 39 / 46; 460^2 x 644, 1 / 2 parts 80 / 92.
    return set(25 * nw <= 7 * W ? 4 : (25 * nw < 18 * W || longest ? 2 : 1), false);
}

int project32_parts(const GeomDev& G, int resident_waves) {
    const long W = resident_waves, nw = G.fwaves, side = std::max(G.rows, G.cols);
    // Through memory where workgroups of several parts leave a tail, as above: 4
    // or 2 in the workgroup / 8 through memory, 1300^2 x 10 angles 80 / 38, x 140
    // 127 / 90, 900^2 x 90 60 / 46, 400^2 x 260 44 / 36; 600^2 x 520 84 / 83.
    if (side > 512 && 8 * nw < 3 * W) return 8;
    if (side >= 380 && (side >= 440 ? 8 : 7) * nw > W && 5 * nw < W) return 8;
    // Four waves per SIMD with four gathers in flight each keep the two-ray
    // form busy: split the rays of grids that stay below that.  Measured, 1 / 2
    // / 4 parts: 64^2 12.5 / 10.7 / 10.8 us, 243^2 x 340 28.8 / 21.0 / 19.7,
    // 300^2 x 424 37.0 / 34.2 / 37.1, 430^2 x 600 62.2 / 61.4 / 69.2, 512^2 x 720
    // 88.3 / 89.5 / 99.9, 2048^2 x 2048 (8 in its place) 2315 / 2318 / 2478.
    if (8 * nw <= W) return WG_PARTS;
    return 2 * nw < W ? 2 : 1;
}

int backproject_tiles(const GeomDev& G, int px) {
    if (G.bp_quad)
        return ((G.cols + G.bp_nq * BPQ_TILE - 1) / (G.bp_nq * BPQ_TILE)) * ((G.rows + BPQ_TILE - 1) / BPQ_TILE);
    return ((G.cols + 8 * px - 1) / (8 * px)) * ((G.rows + BP_TILE - 1) / BP_TILE);
}


int backproject_px(int rows, int cols, int resident_waves) {
    // four pixels per lane amortise more of each angle's work but need more
    // VGPRs: take them when the 4-pixel grid still gives every SIMD four waves
    GeomDev G{};
    G.rows = rows;
    G.cols = cols;
    return (long)backproject_tiles(G, 4) * BP_SPLIT >= resident_waves / 2 ? 4 : 2;
}

// Slack of the candidate windows (pixel units), far above the rounding of the
// window indices.
static double bp_margin(const GeomDev& G) { return 1e-3 + 4e-7 * (double)(G.rows + G.cols + G.nB); }

bool bp_quad_table(const GeomDev& G, const AngleDev* tab, BpAngle* out) {
    const double mg = bp_margin(G);
    const int n = G.cls[2];
    for (int a = n - 1; a >= 0; --a) {
        const AngleDev& A = tab[a];
        const double ac = std::fabs(A.c), as = std::fabs(A.s), S = ac + as;
        const double mn = std::min(ac, as), mx = std::max(ac, as), ds = G.ds;
        // bin q (0, 1, 2) of the block sits at phi + q ds above the block's lower
        // edge, 0 < phi <= ds; A's centre is at mg + S / 2 and its footprint S wide
        if (!(2.0 * S + 2.0 * mg <= 3.0 * ds)) return false;       // the block within three bins
        if (!(S + 2.0 * mg <= 2.0 * ds)) return false;             // A: bin 2 outside
        if (!(0.5 * S + mg < ds)) return false;                    // A: bin 1 above its centre
        if (!(ds <= S)) return false;                              // D: bin 0 outside
        if (!(0.5 * S + mn + mg < 2.0 * ds)) return false;         // B: bin 2 above its centre
        if (!(ds < 0.5 * S + mx)) return false;                    // C: bin 0 below its centre
        if (!(0.5 * S + mx + mg < 2.0 * ds)) return false;         // C: bin 2 above its centre
        if (!out) continue;
        BpAngle& Q = out[a];
        const double inv = A.inv, K = ds * inv;
        Q.cids = A.cids;
        Q.sids = A.sids;
        Q.kb = -(G.s0 + S + mg) / ds + 1.0 + PAD;
        Q.nk = -K;
        Q.wc = (ds - 0.5 * S - mg) * inv;
        Q.einv = A.einv;
        Q.eK = A.einv - K;
        Q.dD1 = (ds - S) * inv;
        Q.dD2 = (2.0 * ds - S) * inv;
        Q.dB0 = -mn * inv;
        Q.dB1 = (ds - mn) * inv;
        Q.eB2 = A.einv - (2.0 * ds - mn) * inv;
        Q.eC0 = A.einv - mx * inv;
        Q.dC1 = (ds - mx) * inv;
        Q.eC2 = A.einv - (2.0 * ds - mx) * inv;
        Q.row = A.row;
        const int code = (A.c < 0.0 ? BP_FLIP_X : 0) | (A.s > 0.0 ? BP_FLIP_Y : 0) |
                         ((A.flags & ANG_HORIZ) ? 0 : BP_VERT);
        const bool same = a + 1 < n && (out[a + 1].run & ((1 << BP_CODE_BITS) - 1)) == code;
        const int end = same ? out[a + 1].run >> BP_CODE_BITS : a + 1;
        Q.run = (end << BP_CODE_BITS) | code;
    }
    return true;
}

void backproject_shape(GeomDev& G, int resident_waves) {
    // Waves of 16 x 16 tiles: enough shares of the angles to fill the wave
    // slots, no more (a share costs its reduction).  Measured, float64 residual
    // form, 4 / 8 / 16 shares: 243^2 x 360 32.7 / 19.7 / 13.6 us, 512^2 x 720
    // 101 / 59 / 61, 1024^2 x 1432 422 / 415 / 410, 2048^2 x 2864 3578 / 3592 /
    // 3729.  Two tiles side by side per wave share an angle's constants but
    // halve the waves: 2048^2 at 4 shares 3.58 -> 3.31 ms, 512^2 slower.
    G.bp_nq = 1;
    const int tiles = backproject_tiles(G, 4);
    G.bp_shares = 12L * tiles < resident_waves ? 16 : (tiles < resident_waves ? 8 : 4);
    G.bp_nq = tiles < resident_waves ? 1 : 2;
}

int project_batch(GeomDev* const* g, int n, int resident_waves) {
    // A batch iteration in us, parts one after another / side by side: 1 x 64^2 96 /
    // 87, 4 x 128^2 130 / 113, 1 x 250^2 164 / 133, 2 x 250^2 (3,900 waves) 197 / 181,
    // 4 x 250^2 259 / 274, 16 x 96^2 (4,700) 144 / 154, 1 x 400^2 (5,000) 259 / 224,
    // 1 x 400^2 x 30 223 / 145; on longer walks the empty slots cost more.
    const long W = resident_waves;
    long waves = 0, steps = 0;
    int most = 0;
    bool uneven = false, any_mem = false;   // among the slices: part counts, sums through memory
    for (int s = 0; s < n; ++s) {
        if (g[s]->parts > WG_PARTS) continue;
        waves += g[s]->nwaves;
        steps += (long)g[s]->nwaves * std::max(g[s]->rows, g[s]->cols);
        uneven |= most && g[s]->parts != most;
        any_mem |= g[s]->pmem != 0;
        most = std::max(most, (int)g[s]->parts);
    }
    const bool side_by_side = 8 * waves <= (steps >= 160 * waves ? 5 : 4) * W;
    // Workgroups of one launch have the waves of the most parts, which slices of
    // fewer leave empty: uneven batches take the parts through memory, in one launch
    // for all slices (144^2 and 386^2: 2 x R 117 -> 92 us).
    const bool mem = side_by_side && (uneven || any_mem);
    for (int s = 0; s < n; ++s)
        if (g[s]->parts <= WG_PARTS) g[s]->pmem = mem ? 1 : 0;
    return side_by_side && !mem ? most : 0;
}

int project_comb_blocks(const GeomDev& G) { return G.nA * ((G.nB + 255) / 256); }

int project_blocks(const GeomDev& G) {
    return G.parts > WG_PARTS ? project_comb_blocks(G) : G.nwg;
}
int project32_blocks(const GeomDev& G) {
    return G.fparts > WG_PARTS ? project_comb_blocks(G) : G.fwg;
}

int build_geometry_into(const sp_geometry* g, int n_cu, GeomDev& G, AngleDev* tab, char* err,
                        size_t errlen) {
    G = GeomDev{};
    G.rows = g->rows;
    G.cols = g->cols;
    G.nA = g->n_angles;
    G.nB = g->n_bins;
    G.xoff = (g->cols - 1) / 2.0;
    G.yoff = (g->rows - 1) / 2.0;
    const double ds = g->bin_spacing / g->pixel;
    const double s0 = (-(g->n_bins - 1) / 2.0 * g->bin_spacing + g->bin_offset) / g->pixel;
    G.ds = ds;
    G.s0 = s0;
    G.inv_ds = 1.0 / ds;
    G.pixel = g->pixel;
    G.pitchX = g->cols + 2 * PAD;
    G.pitchXT = g->rows + 2 * PAD;
    G.pitchB = g->n_bins + 2 * PAD;
    const double margin = bp_margin(G);
    G.nbmax = 1;
    for (int q = 0; q <= 4; ++q) G.cls[q] = 0;
    for (int a = 0; a < g->n_angles; ++a) {
        const AngleDev A = angle_entry(*g, a, ds, s0, margin);
        if (A.nc < 2 || A.nc > 3 || A.nb < 1 || A.nb > 4)
            return geom_fail(err, errlen, "unsupported geometry at angle %d (nc=%d nb=%d)", a, A.nc, A.nb);
        G.nbmax = std::max(G.nbmax, A.nb);
        G.cls[angle_class(A) + 1] += 1;
    }
    for (int q = 1; q <= 4; ++q) G.cls[q] += G.cls[q - 1];
    // stable counting sort by class, no allocation
    int pos[4];
    for (int q = 0; q < 4; ++q) pos[q] = G.cls[q];
    for (int a = 0; a < g->n_angles; ++a) {
        const AngleDev A = angle_entry(*g, a, ds, s0, margin);
        tab[pos[angle_class(A)]++] = A;
    }
    G.pair = 1;
    for (int a = 0; a < G.cls[2]; ++a) G.pair &= pair_fits(G, tab[a]) ? 1 : 0;
    G.nwaves = project_wave_count(G);
    G.nwg = (G.nwaves + 3) / 4;
    G.fwaves = project_pair_waves(G, nullptr);
    G.fwg = (G.fwaves + 3) / 4;
    project_shape(G, n_cu * 32);
    G.fparts = project32_parts(G, n_cu * 32);
    // The blocks sum axis-parallel angles over two candidate bins, which a
    // geometry with oblique angles in blocks never exceeds; one of axis-parallel
    // angles alone has no block to sum.
    G.bp_quad = G.cls[2] > 0 && G.nbmax <= 2 && bp_quad_table(G, tab, nullptr) ? 1 : 0;
    G.bp_px = G.bp_quad ? 4 : backproject_px(g->rows, g->cols, n_cu * 32);
    if (G.bp_quad) backproject_shape(G, n_cu * 32);
    return SP_OK;
}

void bin_sk_fill(const GeomDev& G, double* t) {
    for (int k = -PAD; k < G.nB + PAD; ++k) t[k + PAD] = std::fma((double)k, G.ds, G.s0);
}

namespace {
// A lane's step range as the kernel forms it; false when it is empty (the lane
// then takes no part in its wave's union).
bool lane_steps(const GeomDev& G, const AngleDev& A, int k, int& lo, int& hi) {
    const double sk = std::fma((double)k, G.ds, G.s0);
    if (A.flags & ANG_HORIZ) ray_steps<true>(G, A, sk, lo, hi);
    else ray_steps<false>(G, A, sk, lo, hi);
    return hi > lo;
}
}  // namespace

long wave_steps(const GeomDev& G, const AngleDev* tab, const WaveDev& W) {
    // A wave's lanes hold runs of consecutive bins of one angle.  The rays of an
    // angle that meet the image are consecutive bins, and a ray's range moves
    // monotonically with its bin, so the first and last nonempty ranges of a run
    // bound its union: two rays to evaluate where a lane-by-lane loop took 16 to 64
    // (both forms' tables and orders on one core, 512^2 x 720 13.8 -> 3.7 ms, 243^2 x
    // 360 3.4 -> 1.1; the one-ray form's alone took 15.1 and 3.6).
    int lo = 1 << 30, hi = -1;
    auto add = [&](int ai, int ka, int kb) {
        const AngleDev& A = tab[ai];
        int la, ha, lb, hb;
        bool first = lane_steps(G, A, ka, la, ha), last = lane_steps(G, A, kb, lb, hb);
        // both past the same end of the image: so are those between
        if (!first && !last && la == lb && A.slope != 0.0) return;
        while (!first && ka < kb) first = lane_steps(G, A, ++ka, la, ha);
        if (!first) return;
        while (!last) last = lane_steps(G, A, --kb, lb, hb);
        lo = std::min(lo, std::min(la, lb));
        hi = std::max(hi, std::max(ha, hb));
    };
    if (W.tail == WAVE_ROW) {
        add(W.a0, W.k0, std::min(W.k0 + 63, G.nB - 1));
        return hi > lo ? (long)(hi - lo) : 0;
    }
    // (in units of pairs of bins for the two-ray form)
    const bool pair = W.tail >= WAVE_PAIR_BLOCK;
    const int n = pair ? (G.nB + 1) / 2 : G.nB;
    auto add_units = [&](int ai, int qa, int qb) {
        if (pair) add(ai, 2 * qa, std::min(2 * qb + 1, G.nB - 1));
        else add(ai, qa, qb);
    };
    if (W.tail == WAVE_BLOCK || W.tail == WAVE_PAIR_BLOCK) {
        for (int a = W.a0; a < std::min(W.a0 + WAVE_ANGLES, W.aend); ++a)
            add_units(a, W.k0, std::min(W.k0 + WAVE_BINS, n) - 1);
    } else {
        const int r = n % WAVE_BINS;
        for (int e = W.k0, a = W.a0 + e / r, off = e % r; e < W.k0 + 64 && a < W.aend; ++a, off = 0) {
            const int m = std::min(r - off, W.k0 + 64 - e);
            add_units(a, n - r + off, n - r + off + m - 1);
            e += m;
        }
    }
    return hi > lo ? (long)(hi - lo) : 0;
}

std::vector<int32_t> project_order(const GeomDev& G, const AngleDev* tab, const WaveDev* waves,
                                   int nwaves, int n_cu) {
    const int nwg = (nwaves + 3) / 4;
    std::vector<long> cost((size_t)nwg, 0);
    for (int w = 0; w < nwaves; ++w) cost[(size_t)(w / 4)] += 16 + wave_steps(G, tab, waves[w]);
    std::vector<int32_t> ord((size_t)nwg);
    for (int b = 0; b < nwg; ++b) ord[(size_t)b] = b;
    std::stable_sort(ord.begin(), ord.end(),
                     [&](int32_t x, int32_t y) { return cost[(size_t)x] > cost[(size_t)y]; });
    const int band = std::max(1, n_cu);
    for (int b0 = band, i = 1; b0 < nwg; b0 += band, ++i)
        if (i & 1) std::reverse(ord.begin() + b0, ord.begin() + std::min(nwg, b0 + band));
    return ord;
}

}  // namespace sp
