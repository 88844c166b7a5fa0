// Host check of the forms and launch shapes the library picks for a geometry
// (geometry.cpp), built with AddressSanitizer and UndefinedBehaviorSanitizer on
// the host only.
//
// Input lines: rows cols n_angles n_bins pixel theta0 dtheta bin_spacing
// bin_offset.  Prints one line per geometry; exits 1 at the first violation.
// With the argument "time" (and built with optimisation) it checks instead that
// both forms' wave tables and dispatch orders, which every geometry's set-up
// builds, take at most 1.5 times as long as evaluating the rays of the one-ray table
// lane by lane.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../include/suppcg.h"
#include "../../paper_1807_10151_amd/csrc/sp_internal.h"
#include "../../paper_1807_10151_amd/csrc/sp_walk.h"

using namespace sp;

// R^T's blocks sum the axis-parallel angles over two candidate bins per pixel.
static bool check_blocks(const GeomDev& G, const std::vector<AngleDev>& tab) {
    if (!G.bp_quad) return true;
    for (const AngleDev& A : tab)
        if (A.nb > 2) return std::printf("blocks with %d candidate bins at row %d\n", A.nb, A.row), false;
    return true;
}

// R^T's blocks have one shape, whatever the pixels per lane of the pixel form.
static bool check_tiles(const GeomDev& G) {
    const int gx = G.bp_quad ? BPQ_TILE * G.bp_nq : 8 * G.bp_px, gy = G.bp_quad ? BPQ_TILE : BP_TILE;
    if (backproject_tiles(G, G.bp_px) != ((G.cols + gx - 1) / gx) * ((G.rows + gy - 1) / gy))
        return std::printf("tiles of the default shape\n"), false;
    if (G.bp_quad && backproject_tiles(G, 2) != backproject_tiles(G, 4))
        return std::printf("blocks with 2 pixels per lane\n"), false;
    return true;
}

// R's parts: at most WG_PARTS in one workgroup, which has room for them; on long
// walks only where their grid fills between a half and five eighths of the wave
// slots (their tail costs more than a second launch elsewhere).
static bool check_parts(const GeomDev& G, long W) {
    if (G.parts < 1 || G.parts > 8 || G.fparts < 1 || G.fparts > 8) return std::printf("part counts\n"), false;
    if (!G.pmem && G.parts > WG_PARTS) return std::printf("%d parts in a workgroup\n", G.parts), false;
    if (project_blocks(G) != (G.parts > WG_PARTS ? project_comb_blocks(G) : G.nwg)) return std::printf("partials\n"), false;
    if (G.rows + G.cols > 2 * 512 + 1 && G.parts > 1 && !G.pmem && !(2L * G.nwaves > W && 8L * G.nwaves <= 5 * W))
        return std::printf("%d waves of %dx%d in %d parts in a workgroup\n", G.nwaves, G.rows, G.cols, G.parts), false;
    if (std::max(G.rows, G.cols) > 512 && 8L * G.fwaves < 3 * W && G.fparts <= WG_PARTS)
        return std::printf("%d two-ray waves of %dx%d in %d parts in a workgroup\n", G.fwaves, G.rows, G.cols, G.fparts), false;
    return true;
}

// A batch of n such slices, alone or beside a small one: parts side by side as in the
// slice's own solve while the waves leave slots empty (through memory in one launch
// for all where part counts differ), in sequence once they fill them; more than
// WG_PARTS parts stay as they are.
static bool check_batch(const GeomDev& G, const GeomDev& small, long W) {
    for (int n : {1, 2, 64})
        for (int beside : {0, 1}) {
            std::vector<GeomDev> g((size_t)n, G);
            if (beside) g.push_back(small);
            std::vector<GeomDev*> p;
            long waves = 0;
            bool uneven = false;
            for (GeomDev& q : g) {
                p.push_back(&q);
                if (q.parts <= WG_PARTS) waves += q.nwaves;
                if (q.parts <= WG_PARTS && G.parts <= WG_PARTS && q.parts != G.parts) uneven = true;
            }
            const int wg = project_batch(p.data(), (int)p.size(), (int)W);
            for (const GeomDev& q : g) {
                const GeomDev& was = &q == &g.back() && beside ? small : G;
                if (q.parts != was.parts || (q.parts > WG_PARTS && !q.pmem)) return std::printf("batch of %d: parts\n", n), false;
                if (q.parts > WG_PARTS) continue;
                const bool mem = uneven || (G.parts <= WG_PARTS && G.pmem);
                if (2 * waves <= W && (q.pmem != (mem ? 1 : 0) || wg != (mem ? 0 : q.parts)))
                    return std::printf("batch of %d, %ld waves: %d of %d parts in a workgroup\n", n, waves, wg, q.parts), false;
                if (8 * waves > 5 * W && (wg || q.pmem)) return std::printf("batch of %d, %ld waves: split\n", n, waves), false;
            }
        }
    return true;
}

// Steps of a wave of the one-ray table, every lane's ray evaluated.
static long steps_by_lane(const GeomDev& G, const std::vector<AngleDev>& tab, const WaveDev& W) {
    int lo = 1 << 30, hi = -1;
    for (int lane = 0; lane < 64; ++lane) {
        int ai, k, l, h;
        if (!wave_ray(W, lane, G.nB, ai, k)) continue;
        const AngleDev& A = tab[(size_t)ai];
        if (A.flags & ANG_HORIZ) ray_steps<true>(G, A, bin_pos((double)k, G), l, h);
        else ray_steps<false>(G, A, bin_pos((double)k, G), l, h);
        if (l < h) lo = std::min(lo, l), hi = std::max(hi, h);
    }
    return hi > lo ? hi - lo : 0;
}

static bool check_time(const GeomDev& G, const std::vector<AngleDev>& tab) {
    using clock = std::chrono::steady_clock;
    auto ms = [](clock::duration d) { return std::chrono::duration<double, std::milli>(d).count(); };
    double tables = 1e30, lanes = 1e30;
    long sum = 0;
    std::vector<WaveDev> w((size_t)G.nwaves), f((size_t)G.fwaves);
    for (int r = 0; r < 5; ++r) {
        const auto t0 = clock::now();
        project_waves(G, w.data());
        sum += project_order(G, tab.data(), w.data(), G.nwaves, 256)[0];
        project_pair_waves(G, f.data());
        sum += project_order(G, tab.data(), f.data(), G.fwaves, 256)[0];
        const auto t1 = clock::now();
        for (const WaveDev& W : w) sum += steps_by_lane(G, tab, W);
        const auto t2 = clock::now();
        tables = std::min(tables, ms(t1 - t0));
        lanes = std::min(lanes, ms(t2 - t1));
    }
    for (const WaveDev& W : w)
        if (wave_steps(G, tab.data(), W) != steps_by_lane(G, tab, W)) return std::printf("steps of a wave\n"), false;
    std::printf("tables %.3f ms, lanes %.3f ms (%ld)\n", tables, lanes, sum);
    return tables < 1.5 * lanes;   // (lane by lane the two tables cost more than twice that)
}

int main(int argc, char** argv) {
    const bool timed = argc > 1 && !std::strcmp(argv[1], "time");
    char line[512];
    int count = 0;
    sp_geometry sg{};
    sg.rows = 20, sg.cols = 24, sg.n_angles = 30, sg.n_bins = 35, sg.pixel = sg.bin_spacing = 1.0;
    GeomDev small{};
    std::vector<AngleDev> stab((size_t)sg.n_angles);
    char serr[256] = {0};
    if (build_geometry_into(&sg, 256, small, stab.data(), serr, sizeof serr) != SP_OK) return 1;
    while (std::fgets(line, sizeof line, stdin)) {
        sp_geometry g{};
        if (std::sscanf(line, "%d %d %d %d %lf %lf %lf %lf %lf", &g.rows, &g.cols, &g.n_angles, &g.n_bins, &g.pixel,
                        &g.theta0, &g.dtheta, &g.bin_spacing, &g.bin_offset) != 9)
            continue;
        GeomDev G{};
        std::vector<AngleDev> tab((size_t)g.n_angles);
        char err[256] = {0};
        ++count;
        if (build_geometry_into(&g, 256, G, tab.data(), err, sizeof err) != SP_OK) {
            std::printf("%dx%d %dx%d: refused\n", g.rows, g.cols, g.n_angles, g.n_bins);
            continue;
        }
        if (timed ? !check_time(G, tab) : !check_blocks(G, tab) || !check_tiles(G) || !check_parts(G, 256 * 32) ||
            !check_batch(G, small, 256 * 32)) {
            std::printf("%dx%d %dx%d ds %g: FAILED\n", g.rows, g.cols, g.n_angles, g.n_bins, G.ds);
            return 1;
        }
        std::printf("%dx%d %dx%d ds %g: ok\n", g.rows, g.cols, g.n_angles, g.n_bins, G.ds);
    }
    std::printf("checked %d geometries\n", count);
    return 0;
}
