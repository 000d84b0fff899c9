// Which kernel and tile a GEMM runs on: a function of its shape and the number of CUs alone, in host code without HIP,
// so that it can be asked without a GPU.  jet_gemm.hip launches what plan_gemm returns.
#pragma once

namespace jet {

// the panel kernel's tiles: X(TM, TN, WR, WC, stages, groups per step), 16 TM WR rows x 16 TN WC columns
#define JET_PANELS(X)                                                                                       \
    X(1, 1, 2, 1, 6, 4) X(1, 1, 2, 2, 4, 4) X(2, 1, 1, 3, 3, 4) X(1, 2, 4, 1, 3, 4) X(2, 1, 1, 4, 3, 4)     \
    X(2, 1, 1, 7, 4, 2) X(1, 2, 3, 1, 3, 4) X(1, 2, 3, 2, 5, 2) X(1, 7, 3, 1, 3, 2) X(2, 2, 2, 2, 4, 2)     \
    X(1, 7, 4, 1, 3, 2) X(1, 4, 5, 1, 4, 2) X(1, 7, 5, 1, 3, 2) X(2, 4, 3, 1, 3, 2) X(2, 7, 3, 1, 5, 1)     \
    X(2, 4, 4, 1, 5, 1) X(2, 7, 4, 1, 4, 1)

enum GemmKernel {
    kStrips,         // skinny kernel, 16 columns per workgroup
    kPanel,          // panel kernel, entry `panel` of JET_PANELS
    kTileSmall,      // tile kernel: 128x128, two stages, two workgroups per CU
    kTileSmallDeep,  //              128x128, four stages, one workgroup per CU
    kTileWide,       //              256x128, three stages
    kTileBig,        //              256x256
    kSplitRows,      // two launches: rows [0, split), then the rest, each planned by itself
    kSplitCols       // the same along the columns
};
struct GemmPlan {
    GemmKernel kernel;
    int panel;       // of kPanel
    int bm, bn;      // tile
    long split;      // of kSplit*
};

struct GemmTile {
    int bm, bn;
    GemmKernel kernel;
};
#define JET_PANEL_TILE(TM, TN, WR, WC, S, GP) {16 * TM * WR, 16 * TN * WC, kPanel},
constexpr GemmTile kGemmTiles[] = {JET_PANELS(JET_PANEL_TILE){128, 128, kTileSmallDeep}, {256, 128, kTileWide}, {256, 256, kTileBig}};
#undef JET_PANEL_TILE
constexpr int kNumGemmTiles = sizeof(kGemmTiles) / sizeof(kGemmTiles[0]);
constexpr int kStripPass = 32;       // groups that the skinny kernel chains per pass

constexpr long ceil_div(long a, long b) { return (a + b - 1) / b; }

// The tile of a block-scaled product, by its shape alone: rounds of tiles on the CUs x the time of a tile, which grows
// with its lines per group L = BM + BN as L (L + 550) (measured per group, from HBM, 1 to 4096 rows, 11 matrices:
// 48 lines 0.12 us, 128 lines 0.30, 240 lines 0.62, 384 lines 1.2, 512 lines 1.83).  Over those 140 shapes the choice is
// within 0.7 % of the best tile on average.
inline int pick_tile(long I, long J, long cus, long& rounds) {
    int best = 0;
    long best_cost = -1;
    for (int t = 0; t < kNumGemmTiles; ++t) {
        const GemmTile& c = kGemmTiles[t];
        if (c.bm >= I + 32 && !(c.bm > 128 && I > 100)) continue;         // mostly padding
        if (c.bn == 256 && J % 256) continue;                             // the tile kernel has no ragged columns
        const long r = ceil_div(ceil_div(I, c.bm) * ceil_div(J, c.bn), cus), L = c.bm + c.bn;
        const long cost = r * L * (L + 550);
        if (best_cost < 0 || cost < best_cost) { best = t; best_cost = cost; rounds = r; }
    }
    return best;
}

// Up to 16 rows: the strips of the skinny kernel stream the weights fastest while their passes of 32 groups and the
// CUs' shares of strips are nearly full (28672x4096, 1 row: 26.7 us against 28.7 on panels; 4096x4096 6.1 against 7.1); in a
// partial pass or round waves and CUs wait (55296x5120, 8 and 16 rows: 70 and 78 us, panels 54 and 55; 5120x27648, 1 row:
// 36.7, panels 32).  The part that is full must be 0.7, and 0.9 from 9 rows on, where a strip copies both activation
// blocks (14336x4096, 16 rows: full to 0.875, 17.2 us, panels 14.6).
inline bool strips_keep_busy(long I, long J, long G, long cus) {
    const long strips = J / 16, slots = strips <= cus ? strips : ceil_div(strips, cus) * cus;
    return 10 * G * strips >= (I <= 8 ? 7 : 9) * ceil_div(G, kStripPass) * kStripPass * slots;
}

// OUT[I,J] over G groups of 128.  row_scales: the operand of the columns has a scale per row (WGrad), else per block.
// whole: not a part of a split problem, whose output rows are further apart than the skinny kernel writes them
inline GemmPlan plan_gemm(bool row_scales, long I, long J, long G, long cus, bool whole) {
    if (!row_scales) {
        if (whole && I <= 16 && strips_keep_busy(I, J, G, cus)) return {kStrips, 0, 16, 16, 0};
        // up to 1024 rows, and beyond where one round of tiles does (more rounds: the persistent kernel below, which
        // has no gap between them and splits the last one)
        long rounds = 0;
        const int t = pick_tile(I, J, cus, rounds);
        const GemmTile& c = kGemmTiles[t];
        if ((I <= 1024 || rounds == 1) && c.kernel != kTileSmallDeep) return {c.kernel, t, c.bm, c.bn, 0};
    }
    // the big tile when it divides J and fills the CUs.  The grid is persistent: at most one resident set of
    // workgroups, each walking its tile list.
    const long ti = ceil_div(I, 256), tj = J / 256, big = ti * tj;
    if (J % 256 == 0 && big >= 224) {
        // A last round that fills at most half of the CUs (896 tiles = 3.5 rounds for the 14336-wide
        // WGrads) would cost a whole round: split those tiles off as whole tile rows or tile columns
        // and run them as smaller tiles.  An output element takes the same chain in either kernel.
        const long tail = big % cus;
        if (big > cus && tail > 0 && tail <= cus / 2) {
            if (tail % tj == 0) return {kSplitRows, 0, 256, 256, (ti - tail / tj) * 256};
            if (tail % ti == 0) return {kSplitCols, 0, 256, 256, (tj - tail / ti) * 256};
        }
        return {kTileBig, 0, 256, 256, 0};
    }
    // at most one workgroup per CU anyway: spend the LDS on two more stages, so that operands
    // that come from HBM are fetched three steps ahead
    return {ceil_div(I, 128) * (J / 128) <= cus ? kTileSmallDeep : kTileSmall, 0, 128, 128, 0};
}

}  // namespace jet
