// Host-only check of the covariance build's gather maps (fc_internal.h): for
// every bin count each entry is the one that the record layouts' decoders give
// (f64_tile_at, fp32_pair_at), and filling the largest maps takes well under 20
// ns an entry, best of 20: they are filled on the path of a grid's first build,
// and took 44 ns an entry when every entry decoded its own position.
// Prints "ok" or the first failure.
#include <algorithm>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "fc_internal.h"

using namespace fcx;

int main()
{
    for (int N = 1; N <= 64; ++N) {
        const int ns = n_ksteps(N), P64 = f64_pad(N), P32 = fp32_pad(ns, N);
        std::vector<int16_t> m(cov_maps_size(N, ns), (int16_t)0x7abc);
        cov_maps_fill(N, ns, m.data());
        for (int e = 0; e < f64_sig_double(N); ++e) {
            const int t = 2 * (e >> 5) + (e & 1), pos = (e >> 1) & 15;
            const F64Tile x = f64_tile_at(N, t);
            const int16_t want = t < f64_ntile(N) ? map_w(N, 4 * x.r + (pos & 3) - P64,
                                                          4 * x.kb + (pos >> 2) - P64)
                                                  : kMapZero;
            if (m[e] != want) { printf("N=%d tile entry %d\n", N, e); return 1; }
        }
        const int16_t *m32 = m.data() + 2 * f64_rec_units(N);
        for (int v = 0; v < 4 * n_groups_from_ns(ns); ++v)
            for (int lane = 0; lane < 64; ++lane) {
                const int t = fp32_pair_at(ns, 16 * v + (lane >> 2));
                const int16_t want =
                    t < fp32_npairs(ns) ? map_w(N, 4 * fp32_pair_b(ns, t) + (lane & 3) - P32,
                                                fp32_pair_kp(ns, t) - P32)
                                        : kMapZero;
                if (m32[((v >> 2) * 64 + lane) * 4 + (v & 3)] != want) {
                    printf("N=%d pair entry %d %d\n", N, v, lane);
                    return 1;
                }
            }
    }
    const int ns = n_ksteps(64);
    std::vector<int16_t> m(cov_maps_size(64, ns));
    double best = 1e9;
    for (int k = 0; k < 20; ++k) {
        const auto t0 = std::chrono::steady_clock::now();
        cov_maps_fill(64, ns, m.data());
        best = std::min(best, std::chrono::duration<double, std::nano>(
                                  std::chrono::steady_clock::now() - t0).count());
    }
    if (best / (double)m.size() > 20.0) {
        printf("%.1f ns an entry\n", best / (double)m.size());
        return 1;
    }
    printf("ok\n");
    return 0;
}
