// Host-only check of fixed_plan.h.  Over seeded rounds (group sizes from one to
// thousands, grids from one point to millions) the batches take every row once
// and in order, tiles hold rows of one group and no more than their launch's
// kernel takes, tables stay within the slots, candidate regions are disjoint and
// within their byte bound, and one tile gets a chunk a step; then a round with one group of 20 universes beside
// 2^20 groups of one on 2^20 points, whose candidates took 8.6 GB when every row
// had the most chunks of any launch.
// Prints "ok" or the first failure.
#include <cinttypes>
#include <cmath>
#include <cstdio>
#include <random>
#include <utility>

#include "fixed_plan.h"

using namespace fcx;

static int bad(const char *what, int64_t a = 0, int64_t b = 0)
{
    printf("%s %" PRId64 " %" PRId64 "\n", what, a, b);
    return 1;
}

static int check(const std::vector<int64_t> &m, int64_t G, int64_t slots_max,
                 const int (&resident)[kFxLaunches], int64_t *cand_bytes)
{
    const int64_t R = (int64_t)m.size();
    *cand_bytes = 0;
    for (int64_t r = 0; r < R;) {
        const FxBatch b = fixed_batch(m.data(), r, R, G, 32 * G, slots_max, resident);
        if (b.r_end <= r || b.r_end > R) return bad("batch end", r, b.r_end);
        if ((int64_t)b.slot_m.size() > slots_max) return bad("slots");
        if ((int64_t)b.tiles.size() > kFxMaxTiles) return bad("tiles");
        std::vector<char> seen(b.r_end - r, 0);
        int64_t t = 0, cand = 0;
        for (int k = 0; k < kFxLaunches; ++k) {
            const FxLaunch &l = b.launch[k];
            if (l.tile0 != t) return bad("tile order", k, t);
            if (!l.n_tiles) continue;
            if (l.q_per_chunk % kFxTile || (l.n_chunks - 1) * l.q_per_chunk >= G ||
                l.n_chunks * l.q_per_chunk < G)
                return bad("chunks", l.n_chunks, l.q_per_chunk);
            if (16 * l.rows * l.n_chunks > std::max(kFxCandBytes, 16 * l.rows))
                return bad("candidate bytes", l.rows, l.n_chunks);
            const int lo = k == kFxSmall32 ? 17 : 1;
            const int hi = k == kFxTable ? kFxTile : (k == kFxSmall16 ? 16 : 32);
            for (; t < l.tile0 + l.n_tiles; ++t) {
                const FxTileDesc &td = b.tiles[t];
                if (td.n < lo || td.n > hi) return bad("tile rows", k, td.n);
                if (td.cand0 != cand) return bad("candidates", td.cand0, cand);
                cand += (int64_t)td.n * l.n_chunks;
                for (int64_t x = td.r0; x < td.r0 + td.n; ++x) {
                    if (x < 0 || x >= b.r_end - r || seen[x]++) return bad("row", x);
                    const int64_t want = k == kFxTable ? b.slot_m[td.slot] : td.slot;
                    if (m[r + x] != want) return bad("matrix", m[r + x], want);
                }
            }
        }
        if (cand != b.n_cand) return bad("candidate count", cand, b.n_cand);
        for (char s : seen)
            if (!s) return bad("row left out");
        *cand_bytes = std::max(*cand_bytes, 16 * cand);
        r = b.r_end;
    }
    return 0;
}

int main()
{
    std::mt19937_64 rng(21);
    const auto log_int = [&](double hi) {
        return (int64_t)std::exp(std::uniform_real_distribution<double>(0.0, std::log(hi))(rng));
    };
    int64_t bytes = 0;
    for (int k = 0; k < 400; ++k) {
        std::vector<int64_t> m;
        const int64_t groups = log_int(2000.0);
        const double most = k % 2 ? 3000.0 : 40.0;
        for (int64_t g = 0; g < groups; ++g) m.insert(m.end(), log_int(most), 3 * g + 1);
        const int resident[kFxLaunches] = {512, 512 + 256 * (k % 7), 512 + 512 * (k % 4)};
        if (check(m, log_int(5e6), 1 + log_int(100.0), resident, &bytes)) return 1;
    }
    const int resident[kFxLaunches] = {512, 512, 512};
    std::vector<int64_t> m(20, 0);
    for (int64_t g = 1; g <= (1 << 20); ++g) m.push_back(g);
    if (check(m, 1 << 20, 8, resident, &bytes)) return 1;
    if (bytes > kFxLaunches * kFxCandBytes) return bad("candidates of small groups", bytes);
    // one tile spreads over the chip: a chunk a step on small grids
    const std::vector<int64_t> few(20, 3);
    for (const auto &want : {std::pair<int64_t, int>{64, 1}, {400, 7}, {1600, 25}, {10000, 157}}) {
        const int n = fixed_batch(few.data(), 0, 20, want.first, 512 * want.first, 8, resident).launch[kFxSmall32].n_chunks;
        if (n != want.second) return bad("chunks of one tile", want.first, n);
    }
    // a group of 100: with a table where that is small, without where it is not
    const std::vector<int64_t> hundred(100, 3);
    for (const auto &want : {std::pair<int64_t, int64_t>{32 << 10, 2}, {33 << 10, 0}})
        if (fixed_batch(hundred.data(), 0, 100, 400, want.first, 8, resident)
                .launch[kFxTable].n_tiles != want.second)
            return bad("table of", want.first);
    // one group past the tiles of a batch
    if (check(std::vector<int64_t>(70 << 20, 5), 1000, 8, resident, &bytes)) return 1;
    printf("ok\n");
    return 0;
}
