// Host-only check of scan_geometry.h for large launches: the FP32 and FP64 scans'
// later blocks start beside working ones and a launch waits for part of its last
// chunks, so short chunks in full rounds are chosen; launches of one round cost
// what every block's full start makes them.  Prints "ok" or the first failure.
#include <cinttypes>
#include <cmath>
#include <cstdio>

#include "scan_geometry.h"

using namespace fcx;

int main()
{
    // whole rounds of short chunks were 2, 3.5, 3 and 6 % faster than these many
    // longer ones in rounds less full, or in one
    struct { int64_t tiles, G; int slots; int64_t more_than; ChunkRule rule; } const at[] = {
        {800, 1600, 512, 5, kFp32Chunks},
        {88, 1600, 512, 11, kFp32Chunks},
        {63, 10000, 768, 12, kFp64Chunks},
        {256, 10000, 2048, 8, kPointsChunks},
    };
    for (const auto &a : at) {
        const ScanGeometry g = scan_geometry(a.tiles, a.tiles, a.G, a.slots, a.G, a.rule);
        if (g.n_qchunks <= a.more_than) {
            printf("%" PRId64 " tiles: %" PRId64 " chunks\n", a.tiles, g.n_qchunks);
            return 1;
        }
    }
    for (const ChunkRule &r : {kFp64Chunks, kFp32Chunks, kPointsChunks}) {
        ChunkRule all = r;
        all.later = all.start;
        for (int64_t tiles = 1; tiles < 40; ++tiles)
            for (int64_t c = 1; c <= 100; ++c) {
                const int64_t q = (400 + c - 1) / c, n = (400 + q - 1) / q;
                const bool one = tiles * n <= 512;
                const double a = scan_cost(tiles, 400, 512, r, c), b = scan_cost(tiles, 400, 512, all, c);
                if (one ? a != b : a > b) {
                    printf("%" PRId64 " tiles x %" PRId64 " chunks\n", tiles, c);
                    return 1;
                }
            }
        // every rule's own best count is found
        for (int64_t tiles = 1; tiles < 3000; tiles += 7)
            for (int64_t G : {100, 1600, 10000}) {
                const ScanGeometry g = scan_geometry(tiles, tiles, G, 512, G, r);
                double best = INFINITY;
                const int64_t lo = (G + r.most - 1) / r.most;
                const int64_t hi = std::max(lo, std::min(G / r.least, 2 * lo + 512));
                for (int64_t c = lo; c <= hi; ++c)
                    best = std::min(best, scan_cost(tiles, G, 512, r, c));
                if (g.tried > 51 || scan_cost(tiles, G, 512, r, g.n_qchunks) > best * (1.0 + 1.0 / 32)) {
                    printf("%" PRId64 " tiles x %" PRId64 " points: not the best\n", tiles, G);
                    return 1;
                }
            }
    }
    printf("ok\n");
    return 0;
}
