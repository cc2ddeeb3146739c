// fixed_plan.h -- batches, tiles and grid chunks of the one-matrix scan
// (k_fixed.hip), host code.
//
// The rows of a round (universes in group order, a group being those that share
// a matrix) are taken in batches; a batch's tiles go to three launches: the
// larger groups in tiles of 64 against a t table, the others in tiles of at most
// 32 and 16 that form t on the fly.  Each launch splits the
// grid into its own chunks, and each (row, chunk) leaves a candidate minimum;
// a tile's candidates start at cand0, row by row, n_chunks each.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "scan_geometry.h"

namespace fcx {

constexpr int kFxTile = 64;  // universes per table tile, grid points per step
// Groups up to this size go to k_fixed_small; larger ones share a t table.  The
// table holds 8 G N bytes a group, whose allocation is the larger part of what
// it costs, and the arithmetic per universe crosses near 256 at every N (64
// groups of n universes, the whole call, tables against on the fly: 10 000
// points of 57 bins, n = 100 870 / 658 us, 192 1030 / 954, 256 1158 / 1147; 3600
// of 20 240 / 212, 306 / 301, 331 / 351; 1600 of 64 290 / 329, 381 / 422, 424 /
// 466; 1600 of 12 202 / 175, 264 / 209, 290 / 272).
constexpr int kFxSmall = 256;
// Where a group's table is small, groups of more than one small tile take it (64
// groups of 100, tables against on the fly: 64 points of 4 / 38 / 57 / 64 bins, 2
// to 32 KiB, 137 / 188 / 207 / 235 us against 157 / 211 / 221 / 231; 400 of 4, 12
// KiB, 144 / 163; 400 of 12 and 1600 of 4, 38 and 50 KiB, 182 / 169 and 193 / 169).
constexpr int kFxSmallTable = 32;
constexpr int64_t kFxTableBytes = int64_t(32) << 10;
constexpr int64_t kFxMaxTiles = int64_t(1) << 20;  // tiles of a batch at most
// Candidates of a launch, 16 bytes each, take at most this unless one a row
// takes more: chunks past that bound are not needed to fill the chip.
constexpr int64_t kFxCandBytes = int64_t(64) << 20;

// The launches' chunks, in steps of kFxTile points: as short as one step, since a
// small grid or a late round has few tiles (20 x 20 points of 64 bins, one group
// of 100: 7 chunks 163 us, one 199 us the call).  Start and fill measured over
// 450 calls (4 to 64 bins, 64 to 10 000 points, groups of 8 to 1000, with and
// without iteration): the best of eight pairs; (1, 1), rounds alone, takes 2 %
// longer on average.
constexpr ChunkRule kFxChunks{1, 32, 3.0, 3.0, 0.0, 0.8};

struct FxTileDesc {
    int64_t r0;     // first row (group order) of the tile, in the batch
    int64_t cand0;  // its first candidate
    int32_t n;      // rows in the tile (1..64; k_fixed_small: 1..16 NU)
    int32_t slot;   // matrix slot of the group (k_fixed_small: the matrix's grid point)
};

// One kernel's tiles of a batch and their grid chunks (whole steps of kFxTile
// points).
struct FxLaunch {
    int64_t tile0 = 0, n_tiles = 0, rows = 0, q_per_chunk = 0;
    int n_chunks = 0;
};

enum { kFxTable = 0, kFxSmall16 = 1, kFxSmall32 = 2, kFxLaunches = 3 };

struct FxBatch {
    int64_t r_end = 0;                // the batch's rows end here
    std::vector<int64_t> slot_m;      // matrices of the t tables
    std::vector<FxTileDesc> tiles;    // launch after launch
    FxLaunch launch[kFxLaunches];
    int64_t n_cand = 0;
};

// The batch that starts at row r_begin of R rows whose matrices are m (equal
// ones adjacent): at most slots_max t tables and kFxMaxTiles tiles (a group cut
// by that goes on in the next batch).  table_bytes: of one t table; resident:
// block slots of each launch.
inline FxBatch fixed_batch(const int64_t *m, int64_t r_begin, int64_t R, int64_t G,
                           int64_t table_bytes, int64_t slots_max,
                           const int (&resident)[kFxLaunches])
{
    const int small = table_bytes <= kFxTableBytes ? kFxSmallTable : kFxSmall;
    FxBatch b;
    std::vector<FxTileDesc> part[kFxLaunches];
    int64_t r = r_begin, n_tiles = 0;
    while (r < R && n_tiles < kFxMaxTiles) {
        int64_t r2 = r;
        while (r2 < R && m[r2] == m[r]) ++r2;
        const bool table = r2 - r > small;
        if (table && (int64_t)b.slot_m.size() == slots_max) break;
        FxTileDesc td;
        td.cand0 = 0;
        td.slot = table ? (int32_t)b.slot_m.size() : (int32_t)m[r];
        if (table) b.slot_m.push_back(m[r]);
        for (; r < r2 && n_tiles < kFxMaxTiles; r += td.n, ++n_tiles) {
            td.r0 = r - r_begin;
            td.n = (int32_t)std::min<int64_t>(table ? kFxTile : 32, r2 - r);
            const int k = table ? kFxTable : (td.n > 16 ? kFxSmall32 : kFxSmall16);
            part[k].push_back(td);
            b.launch[k].rows += td.n;
        }
    }
    b.r_end = r;
    const int64_t steps = (G + kFxTile - 1) / kFxTile;
    for (int k = 0; k < kFxLaunches; ++k) {
        FxLaunch &l = b.launch[k];
        l.tile0 = (int64_t)b.tiles.size();
        l.n_tiles = (int64_t)part[k].size();
        if (!l.n_tiles) continue;
        const int64_t most = std::min(steps, std::max<int64_t>(1, kFxCandBytes / (16 * l.rows)));
        const ScanGeometry sg =
            scan_geometry(l.n_tiles, l.n_tiles, steps, resident[k], most, kFxChunks);
        l.q_per_chunk = sg.q_per_chunk * kFxTile;
        l.n_chunks = (int)sg.n_qchunks;
        for (FxTileDesc &td : part[k]) {
            td.cand0 = b.n_cand;
            b.n_cand += (int64_t)td.n * l.n_chunks;
        }
        b.tiles.insert(b.tiles.end(), part[k].begin(), part[k].end());
    }
    return b;
}

}  // namespace fcx
