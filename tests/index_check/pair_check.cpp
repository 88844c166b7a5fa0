// Host check of R's two-ray form (G.pair, sp_walk.h), built with AddressSanitizer
// and UndefinedBehaviorSanitizer on the host only.  For each geometry that takes
// it: the wave table covers every ray exactly once and every wave holds one
// angle class; the wave's step range lies in the image and contains every band
// in which one of its rays meets the image; and in those bands the gathered
// four pixels (the index clamped as the kernel clamps it) with pair_shares
// give each of the two rays the path lengths of the pixels it crosses, from
// clipping the ray against the band directly.
//
// Input lines: rows cols n_angles n_bins pixel theta0 dtheta bin_spacing
// bin_offset ray_stride.  Prints one line per geometry; exits 1 at the first
// violation.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../include/suppcg.h"
#include "../../paper_1807_10151_amd/csrc/sp_internal.h"
#include "../../paper_1807_10151_amd/csrc/sp_walk.h"

using namespace sp;

// Minor-axis interval [u0, u1] (pixel q spans [q, q + 1)) of ray sk in band m.
template <bool HORIZ>
static void band_interval(const GeomDev& G, const AngleDev& A, double sk, int m, double& u0, double& u1) {
    double v[2];
    for (int e = 0; e < 2; ++e) {
        if (HORIZ) {
            const double x = (double)m - G.xoff - 0.5 + e;
            v[e] = G.yoff + 0.5 - (sk - x * A.c) / A.s;
        } else {
            const double y = G.yoff - (double)m + 0.5 - e;
            v[e] = (sk - y * A.s) / A.c + G.xoff + 0.5;
        }
    }
    u0 = std::min(v[0], v[1]);
    u1 = std::max(v[0], v[1]);
}

template <bool HORIZ>
static bool check_pair(const GeomDev& G, const AngleDev& A, int k, int lo, int hi, long& bands, double& worst) {
    const int nmaj = HORIZ ? G.cols : G.rows, nmin = HORIZ ? G.rows : G.cols;
    const int pitch = HORIZ ? G.pitchXT : G.pitchX;
    const bool sw = pair_swap<HORIZ>(A);
    const int kk[2] = {sw ? k + 1 : k, sw ? k : k + 1};   // lower and upper ray
    const double s_lo = bin_pos((double)kk[0], G);
    const double isg = 1.0 / std::fabs(A.slope), delta = pair_delta(G, A);
    double lp = std::fma((double)lo, A.slope, split_b0<HORIZ>(G, A, s_lo));
    for (int m = 0; m < nmaj; ++m) {
        double w[2][8] = {};   // shares of pixels o - PAD .. as the kernel gives them
        int o = 0;
        const bool walked = m >= lo && m < hi;
        if (walked) {
            const unsigned e = std::min((unsigned)(int)lp, (unsigned)(pitch - 4));
            o = (int)e;
            double f, g1, g2;
            pair_shares(lp - std::floor(lp), isg, delta, f, g1, g2);
            w[0][0] = f;
            w[0][1] = 1.0 - f;
            w[1][1] = g1;
            w[1][2] = g2 - g1;
            w[1][3] = 1.0 - g2;
            lp += A.slope;
        }
        for (int r = 0; r < 2; ++r) {
            if (kk[r] >= G.nB) continue;
            double u0, u1;
            band_interval<HORIZ>(G, A, bin_pos((double)kk[r], G), m, u0, u1);
            // rounding of the minor coordinate (a few hundred to a few thousand
            // pixels, advanced step by step), scaled as the shares scale it
            const double tol = (1e-11 + 1e-13 * (G.rows + G.cols)) * (1.0 + isg);
            for (int q = std::max(0, (int)std::floor(u0) - 1); q <= std::min(nmin - 1, (int)std::floor(u1) + 1); ++q) {
                const double want = std::max(0.0, std::min(u1, q + 1.0) - std::max(u0, (double)q)) * isg;
                const int at = q + PAD - o;
                const double got = walked && at >= 0 && at < 4 ? w[r][at] : 0.0;
                worst = std::max(worst, std::fabs(got - want) / tol);
                if (std::fabs(got - want) > tol)
                    return std::printf("row %d bin %d band %d pixel %d: share %.17g, length %.17g\n", A.row, kk[r], m, q,
                                       got, want), false;
            }
            for (int at = 0; walked && at < 4; ++at) {   // no share of a pixel off the ray
                const int q = o + at - PAD;
                if (q < 0 || q >= nmin || (q >= (int)std::floor(u0) - 1 && q <= (int)std::floor(u1) + 1)) continue;
                if (std::fabs(w[r][at]) > tol)
                    return std::printf("row %d bin %d band %d: share of pixel %d off the ray\n", A.row, kk[r], m, q), false;
            }
        }
        ++bands;
    }
    return true;
}

static bool check(const GeomDev& G, const std::vector<AngleDev>& tab, int stride, long& bands, double& worst) {
    std::vector<WaveDev> waves((size_t)G.fwaves);
    if (project_pair_waves(G, waves.data()) != G.fwaves || G.fwg != (G.fwaves + 3) / 4) return std::printf("sizes\n"), false;
    std::vector<unsigned char> seen((size_t)G.nA * G.nB, 0);
    for (const WaveDev& W : waves) {
        const int cls = angle_class(tab[(size_t)W.a0]);
        const bool pair = W.tail == WAVE_PAIR_BLOCK || W.tail == WAVE_PAIR_TAIL;
        if (pair == (cls >= 2)) return std::printf("wave kind %d of class %d\n", W.tail, cls), false;
        const int nmaj = (tab[(size_t)W.a0].flags & ANG_HORIZ) ? G.cols : G.rows;
        int lo = 1 << 30, hi = -1;
        for (int pass = 0; pass < 2; ++pass)
            for (int lane = 0; lane < 64; ++lane) {
                int ai, k;
                if (!(pair ? wave_pair(W, lane, G.nB, ai, k) : wave_ray(W, lane, G.nB, ai, k))) continue;
                if (ai < 0 || ai >= G.nA || k < 0 || k >= G.nB || angle_class(tab[(size_t)ai]) != cls)
                    return std::printf("lane %d: ray (%d, %d)\n", lane, ai, k), false;
                const AngleDev& A = tab[(size_t)ai];
                const bool horiz = A.flags & ANG_HORIZ;
                for (int q = k; pass == 0 && q <= k + (pair ? 1 : 0) && q < G.nB; ++q) {
                    unsigned char& s = seen[(size_t)ai * G.nB + q];
                    if (s) return std::printf("ray (%d, %d) twice\n", ai, q), false;
                    s = 1;
                    int a, b;
                    if (horiz) ray_steps<true>(G, A, bin_pos((double)q, G), a, b);
                    else ray_steps<false>(G, A, bin_pos((double)q, G), a, b);
                    if (a < b) lo = std::min(lo, a), hi = std::max(hi, b);
                }
                if (pass == 0 || !pair || hi <= lo || (((long)ai * G.nB + k) / 2) % stride) continue;
                if (lo < 0 || hi > nmaj) return std::printf("steps [%d, %d) of %d\n", lo, hi, nmaj), false;
                if (!(horiz ? check_pair<true>(G, A, k, lo, hi, bands, worst)
                            : check_pair<false>(G, A, k, lo, hi, bands, worst)))
                    return false;
            }
        if (hi > lo && wave_steps(G, tab.data(), W) != (long)(hi - lo)) return std::printf("host step count\n"), false;
    }
    for (size_t r = 0; r < seen.size(); ++r)
        if (!seen[r]) return std::printf("ray (%zu, %zu) in no wave\n", r / G.nB, r % G.nB), false;
    return true;
}

int main() {
    char line[512];
    int count = 0, taken = 0;
    while (std::fgets(line, sizeof line, stdin)) {
        sp_geometry g{};
        int rs = 1;
        if (std::sscanf(line, "%d %d %d %d %lf %lf %lf %lf %lf %d", &g.rows, &g.cols, &g.n_angles, &g.n_bins,
                        &g.pixel, &g.theta0, &g.dtheta, &g.bin_spacing, &g.bin_offset, &rs) != 10)
            continue;
        GeomDev G{};
        std::vector<AngleDev> tab((size_t)g.n_angles);
        char err[256] = {0};
        ++count;
        if (build_geometry_into(&g, 256, G, tab.data(), err, sizeof err) != SP_OK || !G.pair) {
            std::printf("%dx%d %dx%d ds %g: ray by ray\n", g.rows, g.cols, g.n_angles, g.n_bins, G.ds);
            continue;
        }
        long bands = 0;
        double worst = 0.0;
        if (!check(G, tab, rs, bands, worst)) {
            std::printf("%dx%d %dx%d: FAILED\n", g.rows, g.cols, g.n_angles, g.n_bins);
            return 1;
        }
        std::printf("%dx%d %dx%d ds %g: ok (bands %ld, worst %.2g of the tolerance)\n", g.rows, g.cols, g.n_angles,
                    g.n_bins, G.ds, bands, worst);
        ++taken;
    }
    std::printf("checked %d geometries, %d in pairs\n", count, taken);
    return 0;
}
