// scan_geometry.h -- universe tiles x grid chunks of a scan launch (host code).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace fcx {

// Launch geometry: n_utiles universe tiles, each against n_qchunks grid chunks
// of q_per_chunk points (the last one shorter).
struct ScanGeometry {
    int64_t n_utiles = 0;
    int64_t n_qchunks = 0;
    int64_t q_per_chunk = 0;
    int tried = 0;  // chunk counts looked at: the call's host time
};

// A kernel's chunks, in the units of its grid (points, or steps of several).
// With k of the `resident` blocks that fit on a CU, the CU takes max(fill, k)
// times as long for a unit of all of them as it takes for one block's unit at
// full rate, and `start` such units for each block's start (staging its
// universes), or `later` for the blocks that follow others on a CU and start
// while those beside them work; fill is the larger of 2.5 blocks and fill_share
// resident.  Blocks drift apart, and a launch waits for its last one: `spread` of
// a CU's last chunks is added.
struct ChunkRule {
    int64_t least;      // shortest chunk
    int64_t most;       // longest chunk
    double start;
    double later;
    double spread;
    double fill_share;
    int64_t soft_chunks = INT64_MAX;  // more chunks than this cost soft_cost units
    double soft_cost = 0.0;
};

// The scans' chunks are at most 2048 points long, so that the blocks that share
// a chunk stay close and the L2 serves the later readers of each record, and at
// least 4, which spreads a small scan best (300 universes x 100 points of 57
// bins, chunks of 4 against 8 points: FP64 39 against 48 us, FP32 39 against 48
// us).  Start and fill are the best of a sweep over 363 shapes a form (1 to 64
// bins, 100 to 27 000 points, 100 to 8000 universes, up to 20 chunk counts
// each): the counts they choose are on average 2.2 / 0.7 / 0.9 / 0.9 % (FP64 /
// FP32 / split BF16 / FP16) from the best one measured, those of a rule that
// counts rounds of resident blocks alone 14 / 1.7 / 3.8 / 5.2 %, at most 116 %:
// 2000 universes x 400 points of 48 bins in split FP16, 640 blocks 99 us, 248
// blocks 70 us; FP32, 100 universes x 10 000 points of 57 bins, 250 blocks of
// 40 points 117 us, 264 of 38 171 us (eight CUs with two blocks), 500 110 us.
// More FP64 blocks also mean larger partials, hence no more than fill.  The
// points scan, with more blocks a CU, fits whole rounds best.  Launches of many
// rounds set the later starts and the spread (72 shapes a form of 12 000 to
// 204 800 universes, FP64 44 to 100 000; 47 of 1200 to 14 000 grouped by point):
// without them FP64 / FP32 / points were 2.1 / 2.7 / 4.1 % from the best count
// on average, with them 0.5 / 0.3 / 0.6 % (FP32, 22 528 universes x 1600 points of
// 57 bins: 11 chunks 1.25 ms, 23 chunks 1.21 ms; points, 200 x 65 universes x
// 10 000 points of 20 bins: 8 chunks 2.77 ms, 42 chunks 2.60 ms).  Split BF16 /
// FP16 are 0.6 / 0.8 % off; with later starts of 2 3.8 / 6.7 %.
constexpr ChunkRule kFp64Chunks{4, 2048, 15.0, 1.0, 0.06, 0.0},
    kFp32Chunks{4, 2048, 20.0, 2.0, 0.1, 0.8}, kScanChunks{4, 2048, 20.0, 15.0, 0.03, 0.8},
    kPointsChunks{4, 2048, 2.0, 2.0, 0.1, 1.0};

// Time of a launch in c chunks, in units of one block's unit at full rate: whole
// rounds of resident blocks, and a last one that the CUs share out.
inline double scan_cost(int64_t tiles, int64_t G, int slots, const ChunkRule &rule, int64_t c)
{
    const int64_t cus = slots < 256 ? slots : 256;
    const int64_t q = (G + c - 1) / c, n = (G + q - 1) / q;
    const int64_t resident = slots / cus, blocks = tiles * n;
    const int64_t rounds = blocks / slots, last = (blocks - rounds * slots + cus - 1) / cus;
    const double fill = std::max(2.5, rule.fill_share * (double)resident);
    const auto work = [&](int64_t k) { return k ? (double)q * std::max(fill, (double)k) : 0.0; };
    const int64_t first = rounds ? resident : last;  // blocks of a CU that start together
    const int64_t after = rounds * resident + last - first;
    return (double)rounds * work(resident) + work(last) + rule.start * (double)first +
           rule.later * (double)after + rule.spread * work(last ? last : resident) +
           (n > rule.soft_chunks ? rule.soft_cost : 0.0);
}

// n_utiles tiles of which about `tiles` have work, G grid units, `slots`
// resident blocks, at most max_chunks chunks: the count of the least scan_cost.
// All blocks of a launch take about the same time, one chunk each, so a round
// that is not full is lost (FP64, 1000 tiles x 10 000 points on 768 slots: 5
// chunks in 6.5 rounds 67.6 ms, 23 in 29.95 rounds 65.2 ms; split FP16, 20 tiles
// x 216 000 points on 512 slots: 106 chunks in 4.1 rounds 12.7 ms, 128 in 5.0
// rounds 11.0 ms).  The best count is an end of the range or the most chunks
// that j blocks a CU hold, and what a last round loses matters little once j is
// large, so that 48 values of j are tried (all counts took 1 us more on the host
// at 2500 points, 4 us at 2^20 and 14 us at 2^22).
inline ScanGeometry scan_geometry(int64_t n_utiles, int64_t tiles, int64_t G, int slots,
                                  int64_t max_chunks, const ChunkRule &rule)
{
    constexpr int64_t kTry = 48;
    ScanGeometry sg;
    sg.n_utiles = n_utiles;
    tiles = std::max<int64_t>(tiles, 1);
    // blocks x 256 work-items stay well inside the 32-bit dispatch size
    const int64_t fit = (int64_t(1) << 23) / std::max<int64_t>(n_utiles, 1);
    const int64_t cap = std::max<int64_t>(1, std::min(max_chunks, fit));
    const int64_t lo = std::min(cap, (G + rule.most - 1) / rule.most);
    const int64_t hi = std::min(cap, std::max(lo, std::min(G / rule.least, 2 * lo + 512)));
    double best = 0.0;
    const auto look = [&](int64_t c) {
        if (c < lo || c > hi) return;
        const double cost = scan_cost(tiles, G, slots, rule, c);
        if (sg.tried++ == 0 || cost < best) {
            best = cost;
            sg.q_per_chunk = (G + c - 1) / c;
        }
    };
    const int64_t cus = slots < 256 ? slots : 256;
    const int64_t j0 = (tiles * lo + cus - 1) / cus, j1 = (tiles * hi + cus - 1) / cus;
    look(lo);
    look(rule.soft_chunks);
    if (tiles < cus)
        for (int64_t j = j0; j <= j1 && j < j0 + kTry; ++j) look(j * cus / tiles);
    else  // every count is some j's
        for (int64_t c = lo + 1; c < hi && c < lo + kTry; ++c) look(c);
    look(hi);
    sg.n_qchunks = (G + sg.q_per_chunk - 1) / sg.q_per_chunk;
    return sg;
}

// The scan of universes grouped by true point gives tile t to XCD (t / 8) mod 8
// (k_scan_pts.hip) and an XCD's blocks stay there, so that a launch lasts as long
// as its fullest XCD: the tiles that eight of those would hold (60 tiles: 64; 20
// x 700 universes x 2500 points of 57 bins in 17 chunks on 1024 slots, 136 blocks
// for an XCD's 128 slots, 1.32 ms, in 16 chunks 1.17 ms).
inline int64_t pts_busy_tiles(int64_t tiles)
{
    if (tiles <= 0) return 0;
    const int64_t groups = (tiles + 7) / 8, per_xcd = (groups + 7) / 8;
    const int64_t last = groups - 8 * (per_xcd - 1);  // groups of the last sweep over the XCDs
    return 8 * (last > 1 ? 8 * per_xcd : 8 * (per_xcd - 1) + tiles - 8 * (groups - 1));
}

}  // namespace fcx
