// Host-only check of scan_geometry.h.  Over seeded shapes (tiles, grid sizes
// and resident blocks from one to the largest) and every rule:
//   - the chunks cover the grid once, within the least length, the count's
//     limits and the dispatch size;
//   - the choice costs at most 1/32 more than the best of all counts, and only
//     a few counts were looked at;
// then shapes that a rule of whole rounds slows down, and pts_busy_tiles against
// the tiles that block b = xcd + 8 (m + 8 (j + J c)) is given.
// Prints "ok" or the first failure.
#include <cinttypes>
#include <cmath>
#include <cstdio>
#include <random>

#include "scan_geometry.h"

using namespace fcx;

static int check(int64_t n_utiles, int64_t tiles, int64_t G, int slots, int64_t max_chunks,
                 const ChunkRule &rule)
{
    const ScanGeometry g = scan_geometry(n_utiles, tiles, G, slots, max_chunks, rule);
    const auto bad = [&](const char *what) {
        printf("%s: tiles %" PRId64 "/%" PRId64 " G %" PRId64 " slots %d max %" PRId64
               " least %" PRId64 " -> %" PRId64 " x %" PRId64 " after %d\n",
               what, tiles, n_utiles, G, slots, max_chunks, rule.least, g.n_qchunks,
               g.q_per_chunk, g.tried);
        return 1;
    };
    const int64_t n = g.n_qchunks, q = g.q_per_chunk;
    if (g.n_utiles != n_utiles || n < 1 || q < 1) return bad("empty");
    if (n * q < G || (n - 1) * q >= G) return bad("cover");
    if (n > std::max<int64_t>(max_chunks, 1)) return bad("count");
    if (n > 1 && n * n_utiles > (int64_t(1) << 23)) return bad("dispatch");
    const int64_t cap = std::max<int64_t>(
        1, std::min(max_chunks, (int64_t(1) << 23) / std::max<int64_t>(n_utiles, 1)));
    const int64_t lo = std::min(cap, (G + rule.most - 1) / rule.most);
    if (n > 1 && n > lo && q < rule.least) return bad("short chunk");
    if (n > std::max(lo, 2 * lo + 512)) return bad("many chunks");
    if (g.tried > 51) return bad("host time");
    double best = INFINITY;
    const int64_t hi = std::min(cap, std::max(lo, std::min(G / rule.least, 2 * lo + 512)));
    for (int64_t c = lo; c <= hi; ++c) best = std::min(best, scan_cost(tiles, G, slots, rule, c));
    if (scan_cost(tiles, G, slots, rule, n) > best * (1.0 + 1.0 / 32)) return bad("not the best");
    return 0;
}

int main()
{
    std::mt19937_64 rng(20);
    const auto log_int = [&](double hi) {
        return (int64_t)std::exp(std::uniform_real_distribution<double>(0.0, std::log(hi))(rng));
    };
    for (int k = 0; k < 4000; ++k) {
        const int64_t tiles = log_int(8e6), pad = tiles + (k % 3 ? 0 : log_int(64.0));
        const int64_t G = log_int(k % 5 ? 3e5 : 2e9);
        const int slots = 256 * (1 + (int)(rng() % 8));
        const int64_t max_chunks = k % 4 ? G : log_int(1e4);
        ChunkRule f64 = kFp64Chunks;
        f64.soft_chunks = 1 + log_int(1e4);
        f64.soft_cost = 32.0;
        for (const ChunkRule &r : {kScanChunks, kPointsChunks, f64})
            if (G <= 20000000 && check(pad, tiles, G, slots, max_chunks, r)) return 1;
        // the largest grids: the search itself stays short
        if (scan_geometry(pad, tiles, G, slots, max_chunks, kScanChunks).tried > 51) {
            printf("host time at G %" PRId64 "\n", G);
            return 1;
        }
    }
    // 2000 universes x 400 points on split blocks three to a CU: five-point
    // chunks, three blocks a CU, were a quarter slower than one block a CU
    ScanGeometry g = scan_geometry(8, 8, 400, 768, 400, kScanChunks);
    if (8 * g.n_qchunks > 512) { printf("split: %d chunks\n", (int)g.n_qchunks); return 1; }
    // one tile x 10 000 points: no count that gives a few CUs a second block
    for (const ChunkRule &r : {kFp64Chunks, kScanChunks}) {
        g = scan_geometry(1, 1, 10000, 512, 10000, r);
        if (g.n_qchunks > 256 && g.n_qchunks < 400) { printf("%d blocks\n", (int)g.n_qchunks); return 1; }
    }
    // FP64, 2000 universes x 400 points: partials within 2 MiB
    ChunkRule f64 = kFp64Chunks;
    f64.soft_chunks = (2 << 20) / (16 * 2000);
    f64.soft_cost = 32.0;
    g = scan_geometry(16, 16, 400, 1280, 1 << 20, f64);
    if (g.n_qchunks * 16 * 2000 > 2 << 20) { printf("partials of %d\n", (int)g.n_qchunks); return 1; }
    // the tiles of the fullest XCD
    for (int64_t tiles = 1; tiles < 700; ++tiles) {
        const int64_t J = (tiles + 63) / 64;
        int64_t full = 0;
        for (int64_t xcd = 0; xcd < 8; ++xcd) {
            int64_t n = 0;
            for (int64_t j = 0; j < J; ++j)
                for (int64_t m = 0; m < 8; ++m) n += 8 * (xcd + 8 * j) + m < tiles;
            full = std::max(full, n);
        }
        if (pts_busy_tiles(tiles) != 8 * full) {
            printf("tiles %" PRId64 ": %" PRId64 " busy, %" PRId64 " expected\n", tiles,
                   pts_busy_tiles(tiles), 8 * full);
            return 1;
        }
    }
    printf("ok\n");
    return 0;
}
