// Which kernel and tile a GEMM runs on: a function of its shape and the number of CUs alone, in host code without HIP,
// so that it can be asked without a GPU.  jet_gemm.hip launches what plan_gemm returns.
#pragma once

namespace jet {

// the panel kernel's tiles: X(TM, TN, WR, WC, stages, groups per step, ns per group, ns per round), 16 TM WR rows x
// 16 TN WC columns
#define JET_PANELS(X)                                                                              \
    X(1, 1, 2, 1, 6, 4, 123, 1963) X(1, 1, 2, 2, 4, 4, 148, 2247) X(2, 1, 1, 3, 3, 4, 149, 2589)   \
    X(1, 2, 4, 1, 3, 4, 197, 2584) X(2, 1, 1, 4, 3, 4, 209, 2921) X(2, 1, 1, 7, 4, 2, 349, 2700)   \
    X(1, 2, 3, 1, 3, 4, 163, 2459) X(1, 2, 3, 2, 5, 2, 225, 2834) X(1, 7, 3, 1, 3, 2, 404, 3528)   \
    X(2, 2, 2, 2, 4, 2, 287, 2747) X(1, 7, 4, 1, 3, 2, 366, 3886) X(1, 4, 5, 1, 4, 2, 297, 3489)   \
    X(1, 7, 5, 1, 3, 2, 509, 4238) X(2, 4, 3, 1, 3, 2, 361, 3734) X(2, 7, 3, 1, 5, 1, 559, 4527)   \
    X(2, 4, 4, 1, 5, 1, 380, 3826) X(2, 7, 4, 1, 4, 1, 577, 4805)

// Decode kernels (strips, panels): whether the weights are read as lines that are not needed again (`nt`), which leaves the
// 256 MB memory-side cache to the activations and lets more of the stream through: LDS copies from HBM on all CUs 5.5 -> 6.05
// TB/s, on a quarter of them 2.75 -> 2.94.  From 16 MB on, where a model has several times the cache in such
// matrices: a pass over four captured 8B-class layers, 1 row 258 -> 244 us, 32 rows 359 -> 339, 128 rows 394 -> 373.  Below, the
// same within 0.5 % either way (1024x4096 to 4096x3072, 1 to 128 rows).  A matrix that would stay in the memory-side cache between
// calls loses by it, up to half as much again: one matrix over and over, us through the caches -> past them, 5120x27648 16 rows
// 25.2 -> 30.6, 32 rows 26.4 -> 36.4, 64 rows 29.9 -> 43.3; 4096x14336 64 rows 15.5 -> 19.0; 28672x4096 32 rows 19.6 -> 22.9; but
// 14336x4096 1 row 11.2 -> 10.6, and up to 32 MB -1 to +10 %.  Weights read right after they were quantized (18 calls):
// 5120x27648 32 rows 48 -> 33, 4096x14336 32 rows 16.1 -> 13.5, at worst 28672x4096 32 rows 20.7 -> 23.8.  The activations always
// stay in the caches and are read through them.
// Only where the workgroups that share a panel of weights read it together (or one alone does): beside a partly filled row block,
// whose workgroup has fewer lines to wait for, the other one finds nothing in the L2 any more (32-row tiles of 3584x26496, 37 rows
// 31.7 -> 40.0 us; 100x5120x14336 28.9 -> 36.4).  One row block, 1 to 128 rows: 0 to 10 % faster on all of 120 shapes; several
// full ones: 0 to 4 % faster on 53 of 58 (worst 2.7 % slower, 256x7552x5120).  By how much of the last of several blocks is filled
// (114 shapes, 17 to 250 rows of seven matrices, past / through): below a quarter 0.98-1.37 (1.11 on average), below half
// 0.95-1.25 (1.06), below three quarters 0.92-1.12 (0.99), from there on 0.91-1.00 (0.95).  The line could lie at three quarters.
constexpr bool streams_past_the_caches(bool in_step, long J, long R) { return in_step && J * R >= (1L << 24); }

enum GemmKernel {
    kStrips,         // skinny kernel, 16 columns per workgroup
    kPanel,          // panel kernel, entry `panel` of JET_PANELS
    kTileSmall,      // tile kernel: 128x128, two stages, two workgroups per CU
    kTileSmallDeep,  //              128x128, four stages, one workgroup per CU
    kTileHalf,       //              128x64, four stages
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
    int depth = 0;   // of kStrips: units in flight per wave
    bool nt = false; // of kStrips and kPanel: the weights are read past the caches
};

// workgroups of a tile or panel kernel that the CUs hold at a time
constexpr int resident_per_cu(GemmKernel k) { return k == kTileSmall ? 2 : 1; }

struct GemmTile {
    int bm, bn;
    GemmKernel kernel;
    int group, round;    // ns of a group and of a round of tiles on the CUs
};
#define JET_PANEL_TILE(TM, TN, WR, WC, S, GP, GROUP, ROUND) {16 * TM * WR, 16 * TN * WC, kPanel, GROUP, ROUND},
constexpr GemmTile kGemmTiles[] = {JET_PANELS(JET_PANEL_TILE){128, 128, kTileSmallDeep, 643, 3437},
                                   {128, 128, kTileSmall, 1307, 1794}, {256, 128, kTileWide, 885, 4720},
                                   {256, 256, kTileBig, 1732, 7059}, {128, 64, kTileHalf, 511, 2371}};
#undef JET_PANEL_TILE
constexpr int kNumGemmTiles = sizeof(kGemmTiles) / sizeof(kGemmTiles[0]);
constexpr int kNumPanels = kNumGemmTiles - 5;
static_assert(kGemmTiles[kNumPanels].kernel == kTileSmallDeep && kGemmTiles[kNumPanels + 3].kernel == kTileBig, "");
constexpr int kSmallAlone = 1110;    // ns of a group of kTileSmall where only one of a CU's two places is taken
constexpr int kLaunch = 1400;        // ns of a launch
constexpr int kStripPass = 32;       // groups that the skinny kernel chains per pass

constexpr long ceil_div(long a, long b) { return (a + b - 1) / b; }

// n / d for 0 <= n < 2^31, d > 0, without a division, with m = reciprocal(d): 2^32 - d <= m d < 2^32, so n m / 2^32 is below n / d by
// less than 1/2, and its whole part is the quotient or one less.
constexpr unsigned reciprocal(unsigned d) { return 0xffffffffu / d; }
constexpr int quotient(int n, int d, unsigned m) {
    const int q = (int)(((unsigned long long)(unsigned)n * m) >> 32);
    return n - q * d >= d ? q + 1 : q;
}

// Scales of a chunk in the LDS (tile kernel): 16 rows x 4 steps in 256 bytes, blocks of [4 rows][4 steps][4 rows].  Lane l of a copy,
// which writes bytes 4 l .. 4 l + 3, brings step chunk_step(l) of row chunk_row(l); step s of row r is at chunk_place(r) +
// (16 s ^ chunk_swap(r)).  The rows from 8 on have their steps swapped in pairs: the scales of 16 rows, or of 4 x 4
// columns, then lie in 16 of the 32 banks, where rows r and r + 8 would share one.
constexpr int chunk_row(int l) { return 4 * (l >> 4) + (l & 3); }
constexpr int chunk_step(int l) { return ((l >> 2) & 3) ^ (l >> 5); }
constexpr int chunk_place(int r) { return 64 * (r >> 2) + 4 * (r & 3); }
constexpr int chunk_swap(int r) { return 16 * (r >> 3); }

// Time in ns of a launch on tile c, without its fixed part: rounds x (groups x time of a group + a time per round, which is
// ring fill, drain, output and half a launch gap).  The table's times were fitted to every tile on 34 matrices (128 to
// 55296 columns, 256 to 27648 long, 17 to 4096 rows, weights from HBM and from the caches, 2366 shapes), such that the
// choice and not the time comes out right: it was 0.7 % from the best tile on average.  They were fitted before the tile kernel's
// scales travelled in chunks and its steps took their present order, and before the panels read weights past the caches and
// activations first.  On these kernels, activations in the caches: weights from HBM (256 cases, 16 matrices of 1024 to 55296
// columns, 20 to 1000 rows) 1.0 % from the best on average, 10 above 5 %, worst 100x11008x2048 8 % (128x64, not 64x112) and 140
// rows of 5120 columns x 5120 and 27648 6 and 5 % (64x64, not 48x64), and 400 to 700 rows of 4096 to 8192 columns, where 128x128
// tiles with four stages are 4 to 6 % faster than 128x112 panels; from the caches (144 cases) 2.5 %, 27 above 5 %, worst 23 and
// 10 % where the 128x112 panel reads a resident matrix past them (128x27648x5120 35.3 us, 128x128 tiles 28.6; 128x28672x4096 27.7
// and 25.1).  The cost before, rounds x L (L + 550) with L = rows + columns of the tile, had no time per round and took two
// 128x128 tiles of a CU for two rounds.  It was 2.6 % from the best, and short reductions and launches of a few rounds were
// slower than on the kernels before that (us; before, with that cost, now): from HBM 140x16384x1024 12.2, 15.6, 12.0;
// 280x16384x1024 17.1, 20.4, 16.1; 555x28672x4096 120, 126, 96; from the caches 440x4096x4096 17.4, 19.7, 16.7; 1000x5120x27648
// 195, 226, 175.
inline long tile_time(const GemmTile& c, long I, long J, long G, long cus) {
    const long rounds = ceil_div(ceil_div(I, c.bm) * ceil_div(J, c.bn), cus);
    if (c.kernel == kTileSmall)          // the two tiles of a CU run together
        return rounds / 2 * G * c.group + rounds % 2 * G * kSmallAlone + rounds * c.round;
    return rounds * (G * c.group + c.round);
}

// The fastest tile, -1 if none of those that do it in one round (one_round) exists; time: that of the launch.
inline int pick_tile(long I, long J, long G, long cus, bool one_round, long& time) {
    int best = -1;
    for (int t = 0; t < kNumGemmTiles; ++t) {
        const GemmTile& c = kGemmTiles[t];
        if (c.bm > 128 && I <= 128) continue;                             // half of it padding, not measured
        if (c.bn == 256 && J % 256) continue;                             // the tile kernel has no ragged columns
        if (one_round && ceil_div(I, c.bm) * ceil_div(J, c.bn) > resident_per_cu(c.kernel) * cus) continue;
        const long d = tile_time(c, I, J, G, cus);
        if (best < 0 || d < time) { best = t; time = d; }
    }
    return best;
}

// Up to 16 rows: strips of the skinny kernel or panels.  A strip's eight waves share its reduction, a panel's groups come
// one after the other; but in a partly full pass of 32 groups waves wait, and in a partly full round CUs.  Strips against the
// best panel, 1-16 rows, 11 widths of 1024-55296 columns x 8-216 groups (time of strips / time of panels, from HBM):
//  - one pass, all strips resident (at most two per CU): from 14 groups on 0.77-1.05 (320 to 512 strips x 20 to 28 groups up to
//    1.11; from 9 rows on only up to 24 groups).  At 8 to 13 groups (240 cases, 512 to 8192 columns, against the panel of the
//    rule) 0.84-1.01 for up to 256 strips, 0.85-1.06 beyond, the slow ones at 10 to 12 groups: the line at 14 was drawn on the
//    strips before and lies too high by now.
//  - up to 8 rows, at most one strip per CU, more passes: 0.82-1.03 from 36 of 64 groups on.
//  - more strips than CUs and more than two passes: 1.03-1.33.  More than two per CU and 9 rows or more (both activation blocks,
//    one unit in flight per wave): 1.00-1.45.
//  - the rest: passes x rounds full to 0.9: 28672x4096, 1 and 8 rows, 0.86 and 0.86, 8192x8192 0.99 and 1.03; below, 8 rows of 28672
//    columns x 24, 28, 48 and 56 groups 1.11, 1.13, 1.05 and 1.06, 14336x4096 1.03, 8192x6144 1.09.  A line at 0.7, as it was while
//    panels read their weights through the caches, left these (us, 8 rows) at 18.9 for 17.1 and 21.1 for 18.7 (28672x3072, x3584).
inline bool strips_pay(long I, long J, long G, long cus) {
    const bool few = I <= 8;
    const long strips = J / 16, places = strips <= cus ? strips : ceil_div(strips, cus) * cus;
    const long groups = ceil_div(G, kStripPass) * kStripPass;
    if (G <= kStripPass && (strips <= cus || (strips <= 2 * cus && (few || G <= 24)))) return G >= 14;
    if (few && strips <= cus) return 20 * G >= 11 * groups;
    if (strips > cus && G > 2 * kStripPass) return false;
    if (!few && strips > 2 * cus) return false;
    return 10 * G * strips >= 9 * groups * places;
}

// Units in flight per wave of the skinny kernel: three up to a strip per CU, one where all strips are resident two per CU, two (up
// to 8 rows, whose smaller passes leave room for them) beyond.  Times beside the kernel.
inline int strip_depth(long I, long J, long cus) {
    const long strips = J / 16;
    if (strips <= cus) return 3;
    return strips > 2 * cus && I <= 8 ? 2 : 1;
}

// OUT[I,J] over G groups of 128.  row_scales: the operand of the columns has a scale per row (WGrad), else per block.
// whole: not a part of a split problem, whose output rows are further apart than the skinny kernel writes them
inline GemmPlan plan_gemm(bool row_scales, long I, long J, long G, long cus, bool whole) {
    const long ti = ceil_div(I, 256), tj = J / 256, big = ti * tj;
    // A last round of big tiles that fills at most half of the CUs (896 tiles = 3.5 rounds for the 14336-wide
    // WGrads) would cost a whole round: split those tiles off as whole tile rows or tile columns
    // and run them as smaller tiles.  An output element takes the same chain in either kernel.
    const long tail = big % cus;
    GemmPlan split = {kTileBig, 0, 256, 256, 0};
    if (J % 256 == 0 && big > cus && tail > 0 && tail <= cus / 2) {
        if (tail % tj == 0) split = {kSplitRows, 0, 256, 256, (ti - tail / tj) * 256};
        else if (tail % ti == 0) split = {kSplitCols, 0, 256, 256, (tj - tail / ti) * 256};
    }
    if (!row_scales) {
        if (whole && I <= 16 && strips_pay(I, J, G, cus))
            return {kStrips, 0, 16, 16, 0, strip_depth(I, J, cus), streams_past_the_caches(true, J, G * 128)};
        // up to 1024 rows the fastest tile, and beyond where one round of tiles does (more rounds: the persistent kernel
        // below, which has no gap between them and splits the last one)
        long time = 0, rest = 0;
        const int t = pick_tile(I, J, G, cus, I > 1024, time);
        if (t >= 0) {
            if (I <= 1024 && split.kernel != kTileBig) {
                const bool rows = split.kernel == kSplitRows;
                pick_tile(rows ? I - split.split : I, rows ? J : J - split.split, G, cus, false, rest);
                if (tile_time(kGemmTiles[kNumPanels + 3], rows ? split.split : I, rows ? J : split.split, G, cus) + kLaunch + rest < time)
                    return split;
            }
            const GemmTile& c = kGemmTiles[t];
            const bool in_step = I <= c.bm || I % c.bm == 0;
            return {c.kernel, t, c.bm, c.bn, 0, 0, c.kernel == kPanel && streams_past_the_caches(in_step, J, G * 128)};
        }
    }
    // the big tile when it divides J and fills the CUs.  The grid is persistent: at most one resident set of
    // workgroups, each walking its tile list.
    if (J % 256 == 0 && big >= 224) return split;
    // at most one workgroup per CU anyway: spend the LDS on two more stages, so that operands
    // that come from HBM are fetched three steps ahead
    return {ceil_div(I, 128) * (J / 128) <= cus ? kTileSmallDeep : kTileSmall, 0, 128, 128, 0};
}

}  // namespace jet
