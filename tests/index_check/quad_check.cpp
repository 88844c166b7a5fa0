// Host check of R^T's 2 x 2 block form (BpAngle, sp_walk.h), built with
// AddressSanitizer and UndefinedBehaviorSanitizer on the host only.  For each
// geometry that takes it, every (sampled) block of every tile -- partial tiles
// included -- and every oblique angle: each pixel's corner is the one its
// projection says, the weights of the three-bin window equal chord_u at the
// bins' offsets, no bin outside the window (or left out by the pixel's
// corner) has weight, and a window with a crossed bin lies in the padded row.
//
// Input lines: rows cols n_angles n_bins pixel theta0 dtheta bin_spacing
// bin_offset block_stride.  Prints one line per geometry; exits 1 at the first
// violation.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../include/suppcg.h"
#include "../../paper_1807_10151_amd/csrc/sp_internal.h"
#include "../../paper_1807_10151_amd/csrc/sp_walk.h"

using namespace sp;

static bool check(const GeomDev& G, const std::vector<AngleDev>& tab, int stride, long& blocks, double& worst) {
    std::vector<BpAngle> quad((size_t)std::max(1, G.cls[2]));
    if (!bp_quad_table(G, tab.data(), quad.data())) return std::printf("table refused\n"), false;
    for (int a = 0; a < G.cls[2]; ++a) {
        const int end = quad[a].run >> BP_CODE_BITS;
        if (end <= a || end > G.cls[2]) return std::printf("angle %d: run end %d\n", a, end), false;
        for (int e = a; e < end; ++e)
            if (quad[e].run != quad[a].run) return std::printf("angle %d: run of mixed codes\n", a), false;
    }
    const int ni = (G.rows + BPQ_TILE - 1) / BPQ_TILE * BPQ_TILE, nj = (G.cols + BPQ_TILE - 1) / BPQ_TILE * BPQ_TILE;
    long n = 0;
    for (int i0 = 0; i0 < ni; i0 += 2)
        for (int j0 = 0; j0 < nj; j0 += 2) {
            if (n++ % stride) continue;
            ++blocks;
            const double xc = (double)j0 + 0.5 - G.xoff, yc = G.yoff - ((double)i0 + 0.5);
            for (int a = 0; a < G.cls[2]; ++a) {
                const AngleDev& A = tab[(size_t)a];
                const BpAngle& Q = quad[(size_t)a];
                const double kf = bp_quad_kf(xc, yc, Q);
                if (!(std::fabs(kf) < 2e8)) return std::printf("window index %g\n", kf), false;
                const int o = (int)std::floor(kf);
                const double w = bp_quad_w(kf - std::floor(kf), Q);
                double uA[2], uB[3], uC[3], uD[2];
                bp_quad_a(Q, w, uA);
                bp_quad_b(Q, w, uB);
                bp_quad_c(Q, w, uC);
                bp_quad_d(Q, w, uD);
                const double U[4][3] = {{uA[0], uA[1], 0.0}, {uB[0], uB[1], uB[2]}, {uC[0], uC[1], uC[2]},
                                        {0.0, uD[0], uD[1]}};
                double t[4];
                bool seen[4] = {false, false, false, false};
                for (int p = 0; p < 4; ++p) {
                    const int i = i0 + (p >> 1), j = j0 + (p & 1);
                    const double tp = std::fma((double)j - G.xoff, A.c, (G.yoff - (double)i) * A.s);
                    const int corner = bp_quad_corner(Q.run, p);
                    if (corner < 0 || corner > 3 || seen[corner]) return std::printf("corner of pixel %d\n", p), false;
                    seen[corner] = true;
                    t[corner] = tp;
                    const bool inside = i < G.rows && j < G.cols;
                    for (int q = -3; q < 6; ++q) {
                        const double d = bin_pos((double)(o - PAD + q), G) - tp;
                        const double want = chord_u<false>(d, A.einv, A.inv);
                        const double got = q >= 0 && q < 3 ? U[corner][q] : 0.0;
                        // rounding of the offset, scaled as the weight scales it
                        const double tol = 1e-12 * A.inv + 1e-12;
                        worst = std::max(worst, std::fabs(got - want) / tol);
                        if (std::fabs(got - want) > tol)
                            return std::printf("block (%d, %d) angle %d pixel %d bin %d: weight %.17g, chord %.17g\n", i0,
                                               j0, a, p, q, got, want), false;
                        const int k = o - PAD + q;
                        if (inside && want > 0.0 && k >= 0 && k < G.nB && !(o >= 0 && o + 3 <= G.pitchB))
                            return std::printf("block (%d, %d) angle %d: window [%d, %d) leaves the row of %d\n", i0, j0, a,
                                               o, o + 3, G.pitchB), false;
                    }
                }
                if (!(t[0] <= t[1] && t[1] <= t[2] + 1e-12 && t[2] <= t[3]))
                    return std::printf("block (%d, %d) angle %d: corners out of order\n", i0, j0, a), false;
            }
        }
    return true;
}

int main() {
    char line[512];
    int count = 0, taken = 0;
    while (std::fgets(line, sizeof line, stdin)) {
        sp_geometry g{};
        int bs = 1;
        if (std::sscanf(line, "%d %d %d %d %lf %lf %lf %lf %lf %d", &g.rows, &g.cols, &g.n_angles, &g.n_bins,
                        &g.pixel, &g.theta0, &g.dtheta, &g.bin_spacing, &g.bin_offset, &bs) != 10)
            continue;
        GeomDev G{};
        std::vector<AngleDev> tab((size_t)g.n_angles);
        char err[256] = {0};
        ++count;
        if (build_geometry_into(&g, 256, G, tab.data(), err, sizeof err) != SP_OK || !G.bp_quad) {
            std::printf("%dx%d %dx%d ds %g: pixel by pixel\n", g.rows, g.cols, g.n_angles, g.n_bins, G.ds);
            continue;
        }
        long blocks = 0;
        double worst = 0.0;
        if (!check(G, tab, bs, blocks, worst)) {
            std::printf("%dx%d %dx%d: FAILED\n", g.rows, g.cols, g.n_angles, g.n_bins);
            return 1;
        }
        std::printf("%dx%d %dx%d ds %g: ok (blocks %ld, worst %.2g of the tolerance)\n", g.rows, g.cols, g.n_angles,
                    g.n_bins, G.ds, blocks, worst);
        ++taken;
    }
    std::printf("checked %d geometries, %d in blocks\n", count, taken);
    return 0;
}
