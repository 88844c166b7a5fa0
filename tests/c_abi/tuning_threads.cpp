// Threads that update one entry of the launch-shape table: one stores the count of
// the solvers' form, the other that of a float32 image.  Prints how often the first
// found its own count undone.
#include <atomic>
#include <cstdio>
#include <thread>

#include "suppcg.h"

int main() {
    sp_geometry g{};
    g.rows = g.cols = 8;
    g.n_angles = 1;
    g.n_bins = 9;
    g.pixel = g.bin_spacing = 1.0;
    if (sp_tuning_set(&g, 1, 4) != SP_OK) return 2;
    std::atomic<bool> stop{false};
    std::thread other([&] {
        for (int n = 0; !stop; n = (n + 1) % 9) sp_tuning_set32(&g, n);
    });
    int undone = 0;
    for (int i = 0; i < 200000; ++i) {
        const int32_t parts = i % 8 + 1;
        sp_geometry lg;
        int32_t lp = 0, lx = 0, count = 0;
        sp_tuning_set(&g, parts, 4);
        for (int k = 0; k < 4; ++k) {
            sp_tuning_list(&lg, &lp, &lx, 1, &count);
            if (count != 1 || lp != parts) {
                ++undone;
                break;
            }
        }
    }
    stop = true;
    other.join();
    std::printf("%d\n", undone);
    return 0;
}
