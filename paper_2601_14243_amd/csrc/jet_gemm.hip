// Block-scaled FP8 GEMMs  OUT[i,j] = sum_r A[i,r] B[j,r]  (Jet-RL Sec. 2.2: FProp,
// DGrad and WGrad all take this form once both operands are stored with the
// reduction axis contiguous, Table 1; operand granularities of Sec. 4.2).
//
// Every kernel here computes an output element with the chain fixed in
// jet_numerics.h: p_g = one 16x16x128 FP8 MFMA over group g (accumulator input 0),
// s_g = sa*sb, acc = fma(p_g, s_g, acc) for g ascending, bf16 RNE.  p_g does not
// depend on any other group, so kernels are free to compute the p_g of different
// groups wherever they like; only the fma chain is ordered.  That keeps a token
// row bit-identical between decode-shaped and training-shaped calls (Sec. 4.1).
#include <algorithm>
#include <iterator>
#include <mutex>
#include <type_traits>

#include "jet_internal.h"
#include "jet_numerics.h"
#include "jet_plan.h"

namespace jet {

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Lane-linear direct global->LDS copies (no VGPR staging): lane l's 16 (4) bytes land at
// LDS address `lds` + 16 l (4 l).  `lds` and `base` must be wave-uniform.  Written as asm
// so that the copy stays asynchronous: completion is awaited explicitly with
// JET_WAIT_VMCNT + a workgroup barrier before any wave reads the data.
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
}
// kNt: a line that is not needed again (streams_past_the_caches, jet_plan.h)
template <bool kNt = false>
__device__ __forceinline__ void dma16(uint32_t lds, const void* base, uint32_t voff) {
    lds = __builtin_amdgcn_readfirstlane(lds);
    base = uniform_ptr(base);
    if constexpr (kNt)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(lds), "v"(voff), "s"(base)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds), "v"(voff), "s"(base)
                     : "memory");
}
// same, LDS address = lds_base + IMM formed directly in M0 (one scalar instruction)
template <int IMM>
__device__ __forceinline__ void dma16_at(uint32_t lds_base, const void* base, uint32_t voff) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base), "v"(voff), "s"(base), "n"(IMM)
                 : "memory", "scc");
}
__device__ __forceinline__ void dma4(uint32_t lds, const float* ptr) {
    lds = __builtin_amdgcn_readfirstlane(lds);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "s"(lds), "v"(ptr)
                 : "memory");
}

// One MFMA operand fragment from LDS: the lane's two 16-byte pieces.
__device__ __forceinline__ v8i load_frag(const uint8_t* lo, const uint8_t* hi) {
    return make_frag(*reinterpret_cast<const uint4*>(lo), *reinterpret_cast<const uint4*>(hi));
}

// Hardware deals workgroup b to XCD b % 8; give every XCD a contiguous range of
// logical ids so that workgroups sharing operand tiles share an L2.
__device__ __forceinline__ int xcd_contiguous_id(int b, int n) {
    const int x = b & 7, k = b >> 3, q = n >> 3, rem = n & 7;
    return x * q + (x < rem ? x : rem) + k;
}

// ------------------------------------------------------------------------
// Tile kernel.  A workgroup of WI x WJ waves owns a BM x BN output tile
// (BM = WI*TM*16, BN = WJ*TN*16); a wave owns TM x TN MFMA tiles.  Workgroups are
// persistent: each one walks a list of output tiles, and the (tile, group) pairs of
// that list form one continuous stream of steps, so the copy engine, the LDS and the
// matrix core never drain between tiles.
//
// Per step the operand tiles of one group (BM + BN rows x 128 bytes) go global->LDS
// directly as whole cache lines, swizzled so that every fragment ds_read_b128 is
// conflict-free.  S LDS stages (two; three for the 256x128 tile; four for the 128x128 tile when there is at
// most one workgroup per CU); step q lives in stage q % S and is copied S - 1 steps ahead.
//
// Pipeline of one step q, written for S = 2 (t counts the wave's MFMA tiles; `tail` = the last one to three rows of them, which
// tile_schedule says):
//   top      : the column fragments cf[0..TN), the first row fragment and the scales of
//              step q are already in registers (fetched during step q-1)
//   in front of the tail : MFMA stream, row by row; row fragment m+1 is fetched from stage q&1 while row m runs;
//              the scale fmas of tile t-2 run on the VALU under the MFMA of tile t
//   t = first tile of the tail : every LDS read of stage q&1 has returned, the fragments of all tail rows are in registers.  Wait
//              for this wave's copies of step q+1, workgroup barrier.  Now stage (q+1)&1 is complete
//              and stage q&1 is free: start fetching step q+1's fragments and copying step q+2 into stage q&1.
//   tail     : column by column, so that cf[n] is free for step q+1 after every third (second) MFMA
// The only barrier of a step therefore sits in the middle of the MFMA stream, the LDS
// latency of the next step's first fragments hides under the tail of this step,
// and every copy has about one whole step to land.
// With a tail of one row, all waves fetch TN + 1 fragments (80 KB on the 256x256 tile, 500 cycles of the LDS) under their last four
// MFMAs, as many copies as fit go out at once, the A tile's first, and the matrix cores wait for both.  A tail of three rows
// spreads the fetch over twelve MFMAs; the B copies (lines that eight workgroups of an XCD share) go first and the A copies behind
// a gap, since a burst of all eight holds up the LDS reads: with the same tail and no gap 16384x4096x4096 takes as long as
// before.  One row / the schedule now, us: 256x256 block scales 16384x28672x4096 1658 / 1518, 16384x4096x14336 803 / 764,
// 16384x14336x4096 832 / 762, 16384x4096x4096 232 / 217, 1000x14336x4096 62.1 / 56.3, 6016x5120x27648 736 / 710; all A copies of a step
// at its top (late = 4) is 1-2 % faster there on 4096-long reductions and 4 % slower on 14336-long ones from HBM.  256x256 WGrad
// (256 registers: no room for a tail of three) 28672x4096 over 16384 tokens 1886 / 1789, 5120x5120 over 6016 183 / 172.  256x128
// 1024x5120x27648 195 / 180, 700x7168x5120 42.6 / 40.0.  128x128 WGrad 1024x5120 over 16384 tokens 157 / 144, four stages 1024x4096
// 94.5 / 91.  128x128 block scales, one wave per SIMD: waits for its copies and not for the LDS, so a longer tail, which shortens
// their lead, is 1-3 % slower.  Four late copies and not five: 8 shapes with four stages 0 to 2.6 % faster (777x4096x4096 24.5 ->
// 24.0). Two stages, the columns' operand first: 28 shapes 2.3 % faster on average than the rows' first (3619x17280x640 77.3 -> 74.4,
// 7645x5248x2560 135.6 -> 132.8) and none slower by more than 0.4 %, where the rows' operand is in the caches, as the operator in
// front leaves it; from HBM too, 1.7 %, and up to 3.5 % slower where a last round of a few tiles runs alone on its CUs (4821x3456x4608
// 106.9 -> 110.6). 128x64, two late copies and not five: 3.1 to 4.1 % faster on 7 shapes (256x8192x1024 7.82 -> 7.52), the columns'
// operand first alone the same or 1 % slower.  256x256 on one block of rows: 256x55296x5120 91.3 -> 87.2, with its rows from HBM as
// well 94.3 -> 98.7.
// fma lag 3: a wave alone on its SIMD issues an MFMA every 34.5 cycles instead of 39 in a register-only loop, two waves 3 % more of
// them; in the kernel nothing (one wave waits for its copies) or up to 2 % slower.
//
// LDS: S stages [A tile BM*128][B tile BN*128], then two chunks of scales
//   tile: 1 KB block per 8 rows, copied by one instruction that moves 8 whole 128-byte
//         lines (8 consecutive lanes = one line); fragment f (rows 16f..16f+15) = blocks 2f,
//         2f+1.  Row q (0..7) of a block keeps its eight 16-byte chunks at
//         q*128 + 16*(c ^ swz), swz = (row>>1)&7, so the 16 lanes of an MFMA fragment read
//         (rows 0..15, same chunk) hit 16 different 16-byte bank groups: measured 6.4
//         cycles per ds_read_b128 (160 B/clk/CU) against 16.4 for a plain row-major tile
//   scales: a chunk holds four consecutive steps of the stream, copied at the top of every fourth step into one of two buffers for the
//         next four.  256 bytes per 16 rows (jet_plan.h): a copy's lanes read four neighbouring scales of a row together, a step's
//         scales of 16 rows and of four neighbouring columns are conflict-free reads.  With rows r and r + 8 in one bank the
//         reads took 4.2 M cycles more per 16384x4096x4096 launch (SQ_LDS_BANK_CONFLICT; now 0, SQ_WAIT_INST_LDS 20.1 -> 12.0 M) and
//         16384x28672x4096 1691 us instead of 1661, 16384x8192x4096 493 instead of 479.
//         Copied a step at a time, every scale was a request of its own, as many as a third (block scales) or half (WGrad) of the
//         operand lines': us, before -> in chunks: from HBM 1000x4096x14336 82 -> 74, 1024x5120x27648 247 -> 196,
//         1024x5120x5120 53 -> 44, 256x55296x5120 100 -> 93; 16384x28672x4096 1738 -> 1685, 16384x4096x14336 838 -> 785;
//         WGrad 28672x4096 over 16384 tokens 1990 -> 1922, 1024x4096 96 -> 92.  A chunk's addresses take no division
//         (tile origins by reciprocals from the host) and inside a workgroup's last tile a step on: with three divisions per lane
//         and origin, reductions of 2 to 9 groups were 1.6 % slower than with the scales a step at a time (150 shapes from the
//         caches; now 0.1 % faster; us, step at a time, with divisions, now: 257x4096x256 4.48, 4.60, 4.37; 9000x1024x256 11.5,
//         12.0, 11.5; 257x8192x768 7.8, 8.1, 7.7; 600x8192x768 11.4, 11.8, 11.65), from HBM 0.5 % (now 0.4 % faster).
//         What is slower than a step at a time, with the weights in the caches: the 256x128 tile (700x7168x5120 37.8 -> 39.0,
//         1024x5120x27648 175 -> 179) and 128x128 tiles in several rounds (257x49280x2176 53.5 -> 55.6), and on a hot chip (it
//         differs by box) long calls of 16 tile columns (16384x4096x4096 227 -> 231; on another box 223 -> 221).
//         Measured and left out: one piece of a chunk per step (its
//         address in the MFMA stream: 3-5 % slower where one wave runs per SIMD), all operand copies of a step behind its barrier
//         (2-5 % slower on one round of tiles), waits that count the scale copies exactly (7 % slower with four stages), the
//         copies of a chunk inside the MFMA stream, before or behind the operands' (up to 4 % slower, one round 6-14 %), row scales
//         as [16 rows][4 steps] (the same within 0.1 % on average).
// BM = 32 * waves, so every wave copies 4 A blocks per step, and 4 B blocks (BN = 32 * waves) or 2 (BN = 16 * waves,
// block scales only: the 256x128 and the 128x64 tile).
// ------------------------------------------------------------------------

// How a step of the tile kernel is ordered.
struct TileSchedule {
    int tail_rows;   // rows of the wave's MFMA tiles behind the barrier, walked column by column
    int late, gap;   // operand copies issued behind the barrier, one per MFMA, `gap` MFMAs between the B and the A copies
};
template <int SB_MODE, int TM, int S>
constexpr TileSchedule tile_schedule() {
    constexpr bool block = SB_MODE == kSbBlock;
    if (TM == 8) return block ? TileSchedule{3, 6, 5} : TileSchedule{2, 4, 0};                // 256x256
    if (TM == 2) return {1, 2, 0};                                                            // 128x64
    if (S == 3) return {3, 4, 3};                                                             // 256x128
    if (block) return {1, 4, 0};                                                              // 128x128
    return S == 4 ? TileSchedule{3, 4, 0} : TileSchedule{3, 8, 2};
}

template <int SB_MODE, int WI, int WJ, int TM, int TN, int S = 2>
struct TileCfg {
    static constexpr int kWaves = WI * WJ;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int BM = WI * TM * 16, BN = WJ * TN * 16;
    static constexpr int kABytes = BM * 128, kBBytes = BN * 128;
    static constexpr int kBCopies = BN / (8 * kWaves);     // 1 KB blocks of the B tile per wave and step
    static constexpr int kStageBytes = kABytes + kBBytes;
    static constexpr int kStages = S;                    // LDS stages: copies run kStages - 1 steps ahead
    static constexpr int kScaleBytes = BM * 16 + (SB_MODE == kSbBlock ? 256 : BN * 16);   // one chunk of four steps
    static constexpr int kScaleOff = kStages * kStageBytes;
    static constexpr int kLdsBytes = kScaleOff + 2 * kScaleBytes;
    static constexpr int kOccupancy =                    // workgroups per CU: by waves and by LDS
        (512 / kThreads) < (160 * 1024 / kLdsBytes) ? (512 / kThreads) : (160 * 1024 / kLdsBytes);
    static_assert(S >= 2 && kLdsBytes <= 160 * 1024, "stages");
    static_assert(BM == 32 * kWaves && (BN == 32 * kWaves || BN == 16 * kWaves), "copy schedule");
    static_assert(TM % 2 == 0 && TN % 4 == 0, "fragment double buffer and 64-column stores assume even TM and TN a multiple of 4");
};

// Tiles of one persistent workgroup.  The hardware deals workgroup b to XCD b % 8.  The
// logical tile ids are split into 8 contiguous ranges, one per XCD, and the workgroups of
// an XCD take the ids of their range round-robin, so that at any time the workgroups of
// an XCD work on neighbouring ids (8 tile rows x a few tile columns: shared operands,
// one L2).
struct TileList {
    int first, stride, count;   // ids first + k * stride, 0 <= k < count
};
__device__ __forceinline__ TileList tiles_of_workgroup(int b, int n_wg, int n_tiles) {
    const int x = b & 7, j = b >> 3;
    const int wgs_here = (n_wg - x + 7) >> 3;
    const int q = n_tiles >> 3, rem = n_tiles & 7;
    const int start = x * q + (x < rem ? x : rem), n_here = q + (x < rem ? 1 : 0);
    TileList t;
    t.first = start + j;
    t.stride = wgs_here;
    t.count = (j < n_here) ? (n_here - j + wgs_here - 1) / wgs_here : 0;
    return t;
}

template <int SB_MODE, int WI, int WJ, int TM, int TN, int S = 2>
__global__ __launch_bounds__(64 * WI * WJ, 512 / (64 * WI * WJ))
void gemm_tile_kernel(const uint8_t* __restrict__ A, const float* __restrict__ sa,
                      const uint8_t* __restrict__ B, const float* __restrict__ sb,
                      uint16_t* __restrict__ out, int I, int ldo, int R, int tiles_i, int tiles_j, uint32_t band_recip,
                      uint32_t rest_recip) {
    using C = TileCfg<SB_MODE, WI, WJ, TM, TN, S>;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
    const int t = threadIdx.x, w = t >> 6, l = t & 63, r = l & 15, c4 = l >> 4;
    const int G = R / kGroup;

    const TileList mine = tiles_of_workgroup(blockIdx.x, gridDim.x, tiles_i * tiles_j);
    if (mine.count == 0) return;                     // whole workgroup
    const int n_steps = mine.count * G;

    // logical id -> tile origin: bands of 8 tile rows, the last one of the rest, walked column by column
    auto tile_origin = [&](int k, int& i0, int& j0) {
        constexpr int kBand = 8;
        const int lid = mine.first + k * mine.stride, per_band = kBand * tiles_j, rest = tiles_i % kBand;
        const int band = quotient(lid, per_band, band_recip), within = lid - band * per_band;
        const bool whole = band < tiles_i / kBand;
        const int col = whole ? within / kBand : quotient(within, rest, rest_recip);
        i0 = (band * kBand + within - col * (whole ? kBand : rest)) * C::BM;
        j0 = col * C::BN;
    };

    // ---- operand copies: the cursor stands on the step whose tiles are being copied ----
    // Wave w copies the A rows 32w .. 32w+31 and as many or half as many B rows.  Block c holds tile rows
    // 32w + 8c .. + 7; lane l copies 16 bytes of row 32w + 8c + (l>>3): chunk (l&7) ^ swizzle(row),
    // swizzle = (row>>1)&7 = (l>>4) | ((c&1)<<2).
    const uint32_t lane_row = 32 * w + (l >> 3);
    const uint32_t lane_chunk = 16 * ((l & 7) ^ (l >> 4));
    constexpr int kBC = C::kBCopies;
    static_assert(kBC == 4 || (kBC == 2 && SB_MODE == kSbBlock), "per-column scales need 32 columns per wave");
    uint32_t offB[kBC];                 // B rows never run past the end: fixed per-lane offsets
#pragma unroll
    for (int i = 0; i < kBC; ++i)
        offB[i] = (8 * kBC * w + (l >> 3) + 8 * i) * (uint32_t)R + (lane_chunk ^ ((i & 1) * 64));
    const uint8_t *pa, *pb;             // operand tiles of the cursor's step: tile origin + 128 g (wave-uniform)
    int ck, cg, crows;                  // its tile in the list, group, valid A rows of the tile
    auto cursor_at_tile = [&](int k, int i0, int j0) {
        pa = static_cast<const uint8_t*>(uniform_ptr(A + (size_t)i0 * R));
        pb = static_cast<const uint8_t*>(uniform_ptr(B + (size_t)j0 * R));
        ck = k;
        cg = 0;
        crows = I - i0;
    };
    // past the end of the list the cursor stays on the last step (its tiles are then copied again into a stage
    // nobody reads: harmless, and branch-free)
    auto cursor_next = [&]() {
        if (cg + 1 < G) {
            ++cg;
            pa += kGroup;
            pb += kGroup;
        } else if (ck + 1 < mine.count) {
            int i0, j0;
            tile_origin(ck + 1, i0, j0);
            cursor_at_tile(ck + 1, i0, j0);
        }
    };
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane(lds0 + 4 * w * 1024);
    const uint32_t ldsb = __builtin_amdgcn_readfirstlane(lds0 + C::kABytes + kBC * w * 1024);
    constexpr int kCopies = 4 + kBC;
    // copy c of the cursor's step into the stage at LDS offset st: kBC B blocks, 4 A blocks
    auto copy_one = [&](const uint8_t* pa, const uint8_t* pb, int crows, int c, uint32_t st) {
        if (c >= kBC) {
            const int i = c - kBC;
            const uint32_t base = ldsw + st;
            // rows past the end of A repeat the last valid one (their outputs are never stored)
            const uint32_t row = min(lane_row + 8 * i, (uint32_t)(crows - 1));
            const uint32_t off = __umul24(row, (uint32_t)R) + (lane_chunk ^ ((i & 1) * 64));
            switch (i) {
                case 0: dma16_at<0>(base, pa, off); break;
                case 1: dma16_at<1024>(base, pa, off); break;
                case 2: dma16_at<2048>(base, pa, off); break;
                default: dma16_at<3072>(base, pa, off); break;
            }
        } else {
            const uint32_t bbase = ldsb + st;
            switch (c) {
                case 0: dma16_at<0>(bbase, pb, offB[0]); break;
                case 1: dma16_at<1024>(bbase, pb, offB[1]); break;
                case 2: dma16_at<2048>(bbase, pb, offB[kBC > 2 ? 2 : 0]); break;
                default: dma16_at<3072>(bbase, pb, offB[kBC > 2 ? 3 : 0]); break;
            }
        }
    };

    // ---- scale copies: chunks of four consecutive steps of the stream ----
    // Wave w copies the scales of the A rows 32w .. 32w+31, and of as many columns or (every wave the same ones to the same
    // place) the tile's block scales.  Lane l serves step chunk_step(l) of the chunk, which may belong to another
    // tile than its neighbours' steps, of row chunk_row(l) of each 16.
    constexpr int kScaleCopies = SB_MODE == kSbBlock ? 3 : 4;
    const int lstep = chunk_step(l), lrow = chunk_row(l);
    const float* gs[kScaleCopies];
    int sk, chunk_g;                    // tile and group of the chunk's first step
    auto scales_in_tile = [&](int i0, int j0) {          // all steps of the chunk that somebody computes are in the tile at i0, j0
        const int ls = min(lstep, G - 1 - chunk_g);
        const float* a0 = static_cast<const float*>(uniform_ptr(sa + (size_t)i0 * G + chunk_g));
        const float* b0 = static_cast<const float*>(uniform_ptr(sb + (size_t)(SB_MODE == kSbBlock ? j0 >> 7 : j0) * G + chunk_g));
        const int row = 32 * w + lrow, last = I - 1 - i0;
        gs[0] = a0 + (__umul24(min(row, last), G) + ls);
        gs[1] = a0 + (__umul24(min(row + 16, last), G) + ls);
        if (SB_MODE == kSbBlock) {
            gs[2] = b0 + (__umul24(min(lrow, (C::BN + 127) / 128 - 1), G) + ls);
        } else {
            gs[2] = b0 + (__umul24(row, G) + ls);
            gs[kScaleCopies - 1] = b0 + (__umul24(row + 16, G) + ls);
        }
    };
    auto scales_across_tiles = [&]() {                   // this lane's step may belong to a later tile than the chunk's first
        const int st = chunk_g + lstep, dk = (st >= G) + (st >= 2 * G) + (st >= 3 * G), g = st - dk * G, row = 32 * w + lrow;
        int i0, j0;
        tile_origin(min(sk + dk, mine.count - 1), i0, j0);   // past the end of the list: steps nobody computes
        gs[0] = sa + (size_t)min(i0 + row, I - 1) * G + g;
        gs[1] = sa + (size_t)min(i0 + row + 16, I - 1) * G + g;
        if (SB_MODE == kSbBlock) {
            gs[2] = sb + (size_t)((j0 >> 7) + min(lrow, (C::BN + 127) / 128 - 1)) * G + g;
        } else {
            gs[2] = sb + (size_t)(j0 + row) * G + g;
            gs[kScaleCopies - 1] = sb + (size_t)(j0 + row + 16) * G + g;
        }
    };
    auto scales_next = [&]() {
        chunk_g += 4;
        if (chunk_g + 4 <= G || (chunk_g < G && sk + 1 == mine.count)) {   // the last chunk's steps and this one's are in one tile
            const int d = min(4, G - chunk_g + 3 - lstep);                 // steps behind the tile's last one repeat it
#pragma unroll
            for (int i = 0; i < kScaleCopies; ++i) gs[i] += d;
            return;
        }
        while (chunk_g >= G) { chunk_g -= G; ++sk; }
        if (chunk_g + 4 <= G || sk + 1 >= mine.count) {
            int i0, j0;
            tile_origin(min(sk, mine.count - 1), i0, j0);
            scales_in_tile(i0, j0);
        } else {
            scales_across_tiles();
        }
    };
    const uint32_t ldss = __builtin_amdgcn_readfirstlane(lds0 + C::kScaleOff + 32 * w * 16);
    const uint32_t ldst = __builtin_amdgcn_readfirstlane(lds0 + C::kScaleOff + C::BM * 16 + (SB_MODE == kSbBlock ? 0 : 32 * w * 16));
    auto copy_scales = [&](uint32_t buf) {
        dma4(ldss + buf, gs[0]);
        dma4(ldss + buf + 256, gs[1]);
        dma4(ldst + buf, gs[2]);
        if (SB_MODE != kSbBlock) dma4(ldst + buf + 256, gs[kScaleCopies - 1]);
    };

    // ---- fragment addressing ----
    const int wi = w / WJ, wj = w % WJ;
    // this lane's two 16-byte pieces of a fragment (row r, chunks c4 and 4 + c4)
    const int swz = (r >> 1) & 7;
    const int frag_lo = (r >> 3) * 1024 + (r & 7) * 128 + 16 * (c4 ^ swz);
    const int frag_hi = (r >> 3) * 1024 + (r & 7) * 128 + 16 * ((4 + c4) ^ swz);
    auto row_frag = [&](int slot, int m) {
        const uint8_t* p = smem + slot * C::kStageBytes + (wi * TM + m) * 2048;
        return load_frag(p + frag_lo, p + frag_hi);
    };
    auto col_frag = [&](int slot, int n) {
        const uint8_t* p = smem + slot * C::kStageBytes + C::kABytes + (wj * TN + n) * 2048;
        return load_frag(p + frag_lo, p + frag_hi);
    };
    // scales of a step as the lane needs them: sa of its row in each of the TM row tiles and
    // the scale(s) of its columns; off: chunk buffer of the step + 16 * (step & 3)
    // (the per-column scales of WGrad are fetched at the top of the step instead: the
    // first fma needs them two MFMAs later, and there are no registers to hold them early)
    struct RawScales {
        float a[TM];
        float b_block;
    };
    const uint8_t* const sc_rows = smem + C::kScaleOff + wi * TM * 256 + chunk_place(r);
    const uint8_t* const sc_cols = smem + C::kScaleOff + C::BM * 16 + wj * TN * 256 + chunk_place(4 * c4);
    const int swap_row = chunk_swap(r), swap_col = chunk_swap(4 * c4);
    const uint8_t* const sc_block = smem + C::kScaleOff + C::BM * 16 + ((wj * TN * 16) >> 7) * 4;   // one 128-wide block
    auto load_scales = [&](int off, RawScales& s) {
#pragma unroll
        for (int m = 0; m < TM; ++m) s.a[m] = *reinterpret_cast<const float*>(sc_rows + (off ^ swap_row) + m * 256);
        if (SB_MODE == kSbBlock) s.b_block = *reinterpret_cast<const float*>(sc_block + off);
    };
    auto load_col_scales = [&](int off, v4f (&s)[TN]) {
#pragma unroll
        for (int n = 0; n < TN; ++n) s[n] = *reinterpret_cast<const v4f*>(sc_cols + (off ^ swap_col) + n * 256);
    };

    constexpr TileSchedule kSchedule = tile_schedule<SB_MODE, TM, S>();
    constexpr int kTiles = TM * TN, kLag = 2;
    // The scale fmas of tile t-2 run next to the MFMA of tile t, far enough behind their own
    // MFMA that its result needs no wait.  FProp/DGrad: MFMA first, three result buffers.
    // WGrad (twice the VALU work, 16 more registers of column scales): fmas first, two buffers.
    constexpr bool kFmaFirst = (SB_MODE != kSbBlock);
    constexpr int kRing = kFmaFirst ? 2 : 3;
    // MFMA tile t: row by row in front of the barrier, column by column in the kTail rows behind it
    constexpr int kTail = kSchedule.tail_rows, kHead = TM - kTail;
    constexpr int kSync = kHead * TN;                    // the barrier stands behind the MFMA of this tile
    auto tile_row = [](int t) { return t < kSync ? t / TN : kHead + (t - kSync) % kTail; };
    auto tile_col = [](int t) { return t < kSync ? t % TN : (t - kSync) / kTail; };
    // Buffer of a row's fragment: two take turns, and the rows behind the barrier beyond the first have one each.  That first row
    // takes the buffer that the last row in front of the barrier does not have, and the next step's row 0, fetched behind the
    // barrier, takes the other one: the last row in front of it has row 0's, so where their number is even, row 2 goes elsewhere.
    static_assert(kHead % 2 == 1 || (kHead >= 6 && kTail >= 2), "row 2's buffer is free again when it is needed");
    auto row_buf = [](int m) { return m > kHead ? m - kHead + 1 : kHead % 2 ? m & 1 : m < 3 ? m : (m - 3) & 1; };
    constexpr int kLate = kSchedule.late;                // operand copies issued behind the barrier, the rest at the top of the next step
    auto late_copy = [](int t) {                         // the one behind the MFMA of tile t, -1 if none
        const int v = t - kSync - 1, c = v < kBC ? v : v - kSchedule.gap;
        return v >= 0 && (v < kBC || c >= kBC) && c < kLate ? c : -1;
    };
    static_assert(kLate >= 1 && kLate <= kCopies && kCopies - kLate <= kSync, "copy slots");
    static_assert(kSync + kLate + (kLate > kBC ? kSchedule.gap : 0) < kTiles + kLag, "copy slots");

    // Vector-memory operations of a wave in step j, in their order: at the top of every fourth step the scales of chunk
    // j / 4 + 1, the rest of the operand copies of step j + S - 1 (none where all are late), behind the barrier the first kLate
    // operand copies of step j + S, behind a tile's last step its stores.  The scales of chunk c (steps 4c .. 4c + 3) are issued at
    // the top of step 4c - 4 and first read behind the barrier of step 4c - 1, which waits for the operands of step 4c.  The last
    // copy of those is issued at the top of step 4c + 1 - S >= 4c - 3, or, where all are late, behind the barrier of step
    // 4c - S >= 4c - 4: behind the scales in either case.  Their buffer held chunk c - 2, last read in step 4c - 5.
    constexpr int kYounger = (S - 2) * kCopies;      // at the barrier of step q, behind the copies of step q + 1 (at least)
    // ---- prologue: chunk 0, operands of steps 0 .. S - 1 (of the last the first kLate) ----
    int first_i0, first_j0;
    tile_origin(0, first_i0, first_j0);
    cursor_at_tile(0, first_i0, first_j0);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) copy_one(pa, pb, crows, i, 0);
    sk = chunk_g = 0;
    if (G >= 4 || mine.count == 1) scales_in_tile(first_i0, first_j0);
    else scales_across_tiles();
    copy_scales(0);
#pragma unroll 1
    for (int s = 1; s < S - 1; ++s) {
        cursor_next();
#pragma unroll
        for (int i = 0; i < kCopies; ++i) copy_one(pa, pb, crows, i, (uint32_t)(s * C::kStageBytes));
    }
    cursor_next();
#pragma unroll
    for (int i = 0; i < kLate; ++i) copy_one(pa, pb, crows, i, (uint32_t)((S - 1) * C::kStageBytes));
    JET_WAIT_VMCNT((S - 2) * kCopies + kLate);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    v8i cf[TN], xf[kTail + 1];
    RawScales next;
#pragma unroll
    for (int n = 0; n < TN; ++n) cf[n] = col_frag(0, n);
    xf[0] = row_frag(0, 0);
    load_scales(0, next);
    // s = sa * sb of the coming step (block scales: one binary32 product per row tile), formed as
    // soon as the scales are in, so that the top of a step never waits for the LDS
    float sai_n[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) sai_n[m] = (SB_MODE == kSbBlock) ? next.a[m] * next.b_block : next.a[m];

    v4f acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    int sc_off = 0;                     // where the scales of step q are, from the first buffer
    for (int q = 0, k = 0, g = 0; q < n_steps; ++q) {
        const int slot = ((S & (S - 1)) == 0) ? (q & (S - 1)) : (q % S);
        const int nslot = (slot + 1 == S) ? 0 : slot + 1;
        const int oslot = (slot == 0) ? S - 1 : slot - 1;   // of step q+S-1
        const uint32_t st_this = __builtin_amdgcn_readfirstlane(slot * C::kStageBytes);
        const uint32_t st_other = __builtin_amdgcn_readfirstlane(oslot * C::kStageBytes);
        // all control flow of a step is here
        if ((q & 3) == 0 && q + 4 < n_steps) {
            scales_next();
            copy_scales((q & 4) ? 0 : C::kScaleBytes);
        }
        const uint8_t *pa0 = pa, *pb0 = pb;         // the rest of step q + S - 1 is copied first
        const int crows0 = crows;
        cursor_next();                              // step q + S
        int sc_next = sc_off + 16;
        if ((q & 3) == 3) sc_next = (q & 4) ? 0 : C::kScaleBytes;

        // ---- one straight-line block from here to the end of the tile loop ----
        // scales of this step: s = sa * sb, one binary32 product per (row, column scale)
        float sai[TM];
        v4f sbj[TN];
#pragma unroll
        for (int m = 0; m < TM; ++m) sai[m] = sai_n[m];
        if (SB_MODE != kSbBlock) load_col_scales(sc_off, sbj);

        v4f pr[kRing];
#pragma unroll
        for (int t = 0; t < kTiles + kLag; ++t) {
            auto scale_fmas = [&]() {
                if (t < kLag) return;
                const int u = t - kLag, m = tile_row(u), n = tile_col(u);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = (SB_MODE == kSbBlock) ? sai[m] : sai[m] * sbj[n][e];
                    acc[m][n][e] = chain(pr[u % kRing][e], s, acc[m][n][e]);
                }
            };
            if (kFmaFirst) {
                scale_fmas();
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t < kTiles) {
                const int m = tile_row(t), n = tile_col(t);
                pr[t % kRing] = group_product(cf[n], xf[row_buf(m)]);
                // next row's fragment, fetched behind the MFMA: a fetch in front of it would be
                // included in whatever LDS wait that MFMA's operands need
                __builtin_amdgcn_sched_barrier(0);
                if (t < kSync && n == 0) xf[row_buf(m + 1)] = row_frag(slot, m + 1);
                // those of the other rows behind the barrier, a row earlier where there is one
                constexpr int kOthers = (kHead > 2 ? kHead - 2 : 0) * TN + 1;
                if (t >= kOthers && t < kOthers + kTail - 1) {
                    const int row = kHead + 1 + t - kOthers;
                    xf[row_buf(row)] = row_frag(slot, row);
                }
            }
            if (!kFmaFirst) scale_fmas();
            __builtin_amdgcn_sched_barrier(0);
            if (t == kSync) {
                // every read of stage `slot` has returned: the MFMA above needed the last one, or it is waited for;
                // of this wave's copies only those of steps q+2 .. q+S-1 may still be on their way
                if (kTail > 1) __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
                JET_WAIT_VMCNT(kYounger);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                xf[0] = row_frag(nslot, 0);
                load_scales(sc_next, next);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t == kTiles - 1) {
                // the scales fetched after the barrier are in by now (only later fetches are still out)
#pragma unroll
                for (int m = 0; m < TM; ++m) sai_n[m] = (SB_MODE == kSbBlock) ? next.a[m] * next.b_block : next.a[m];
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t >= kSync && t < kTiles && tile_row(t) == TM - 1) {
                cf[tile_col(t)] = col_frag(nslot, tile_col(t));      // its last MFMA of this step is issued
                __builtin_amdgcn_sched_barrier(0);
            }
            if (late_copy(t) >= 0) {
                copy_one(pa, pb, crows, late_copy(t), st_this);           // step q+S goes into stage `slot`
                __builtin_amdgcn_sched_barrier(0);
            } else if (t < kCopies - kLate) {
                copy_one(pa0, pb0, crows0, kLate + t, st_other);          // remaining copies of step q+S-1
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        sc_off = sc_next;
        if (++g < G) continue;
        g = 0;

        // epilogue of tile k.  A lane holds row r, columns 4 c4 .. 4 c4 + 3 of each MFMA tile.  Two
        // row-swaps between neighbouring column tiles give every lane 8 consecutive columns
        // (16 bytes) and the four lanes of a row 64 contiguous bytes; exchanging the upper eight
        // rows of one such pair of tiles with the lower eight rows of the next pair then gives
        // every row a whole 128-byte line per store instruction (8 rows x 128 B instead of
        // 16 rows x 64 B: half as many memory transactions).
        int i0, j0;
        tile_origin(k, i0, j0);
        const bool upper = (r & 8) != 0;
#pragma unroll
        for (int m = 0; m < TM; ++m) {
#pragma unroll
            for (int n = 0; n < TN; n += 4) {
                uint32_t lo[4], hi[4];   // this lane's 16 bytes of column tiles n, n+1 and of n+2, n+3
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int nn = n + 2 * half;
                    const uint32_t a0 = bf16_pack2(acc[m][nn][0], acc[m][nn][1]);
                    const uint32_t a1 = bf16_pack2(acc[m][nn][2], acc[m][nn][3]);
                    const uint32_t b0 = bf16_pack2(acc[m][nn + 1][0], acc[m][nn + 1][1]);
                    const uint32_t b1 = bf16_pack2(acc[m][nn + 1][2], acc[m][nn + 1][3]);
                    // lanes 16-31 and 48-63 of the first operand <-> lanes 0-15 and 32-47 of the second
                    const auto s0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
                    const auto s1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
                    uint32_t* d = half ? hi : lo;
                    d[0] = s0[0]; d[1] = s1[0]; d[2] = s0[1]; d[3] = s1[1];
                    acc[m][nn] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    acc[m][nn + 1] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                }
                uint4 first, second;     // rows 0-7 / rows 8-15 of the row tile, 64 columns each
                uint32_t* f = &first.x;
                uint32_t* g2 = &second.x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // row_ror:8 swaps the two halves of every 16-lane row: lane r sees lane r ^ 8
                    const uint32_t hi_x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi[e], 0x128, 0xf, 0xf, true);
                    const uint32_t lo_x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo[e], 0x128, 0xf, 0xf, true);
                    f[e] = upper ? hi_x : lo[e];
                    g2[e] = upper ? hi[e] : lo_x;
                }
                const int jc = j0 + (wj * TN + n + (c4 & 1)) * 16 + (c4 >> 1) * 8 + (upper ? 32 : 0);
                const int ia = i0 + (wi * TM + m) * 16 + (r & 7);
                if (ia < I) *reinterpret_cast<uint4*>(out + (size_t)ia * ldo + jc) = first;
                if (ia + 8 < I) *reinterpret_cast<uint4*>(out + (size_t)(ia + 8) * ldo + jc) = second;
            }
        }
        ++k;
    }
    JET_WAIT_VMCNT(0);   // nothing may be in flight towards the LDS when it is released
}

// ------------------------------------------------------------------------
// Skinny kernel for I <= 16 (decode): bound by streaming B (the weights) once.
// A workgroup of kSkWaves waves owns 16 output columns and the whole reduction.  The
// groups of a pass (32 groups) are dealt to the waves in runs of four consecutive
// groups, those of a last, partial pass evenly; every wave streams its own units (16 weight rows + the rows of the batch's
// 8-row blocks of one group) through a private LDS ring with kSkDepth units in flight, and the scales of a run at once,
// using the same whole-line LDS-DMA and swizzled fragment layout as the tile kernel --
// no barrier is needed for the ring.  After every pass the p_g and s_g meet in LDS and
// four waves run the ordered fma chain for their quarter of the outputs.
// A CU has about 320 lines in flight, and every 4-byte scale fetched on its own costs one: with the scales of four groups in one
// copy, partial passes dealt evenly and (up to 8 rows, more than one round of strips) a second unit in flight per wave,
// for which only the batch's rows of a group meet in the LDS, from HBM, us, before -> now: 28672x4096 1 row 25.1 -> 22.3, 8 rows
// 25.9 -> 22.6; 14336x4096 1 row 14.5 -> 13.6; 4096x14336 1 row 14.7 -> 14.3; 6144x2048 1 row 6.4 -> 5.6; 4096x4096 16 rows
// 7.1 -> 6.7; 1024x4096 1 row 5.4 -> 5.1.  With two units in flight where all strips are resident, 8 rows of 6144x4096 take 8.5
// instead of 7.9.
// ------------------------------------------------------------------------
constexpr int kSkPass = kStripPass;               // groups chained per pass
template <int kDepth, int kWaves, int ABLK>
struct SkinnyCfg {
    // rows of the output that meet in the LDS: all 16, or with two units in flight and two workgroups per CU those of the block
    static constexpr int kRows = kDepth == 2 ? 8 * ABLK : 16;
    static constexpr int kUnit = 2048 + 1024 * ABLK;                 // weight fragment, activation fragment of a group
    static constexpr int kScales = 256 * ABLK;                       // scales of a run of four groups: [row][4], then the block's
    static constexpr int kRing = kDepth * kUnit + 2 * kScales;       // of a wave
    static constexpr int kGroupBytes = 20 * kRows * 4;                // p[4][4][kRows], s[4][kRows]
    static constexpr int kLds = kWaves * kRing + kSkPass * kGroupBytes;
};

// kSkDepth = units in flight per wave: 3 when there is at most one workgroup per CU, 1 or 2 when the strips outnumber the CUs (two
// workgroups then share a CU and cover each other's start-up, chain passes and drain)
// kSkWaves = waves splitting the groups of a strip
// ABLK = 8-row blocks of activations that hold a row of the batch ((I + 7) / 8): only these are
// copied, and of the last one only the lines of existing rows -- every byte through a CU's
// memory pipeline costs the same there whether it misses or hits, so at I = 1 the copy of 15
// repeated rows would double the time of a strip.  The fragments of the other rows are read from
// LDS that no copy wrote; their products land in output rows that are never stored.
template <int kSkDepth, int kSkWaves, int ABLK>
__global__ __launch_bounds__(64 * kSkWaves) void gemm_skinny_kernel(const uint8_t* __restrict__ A,
                                                                     const float* __restrict__ sa,
                                                                     const uint8_t* __restrict__ B,
                                                                     const float* __restrict__ sb,
                                                                     uint16_t* __restrict__ out, int I, int J,
                                                                     int R, bool nt) {
    using C = SkinnyCfg<kSkDepth, kSkWaves, ABLK>;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
    const int t = threadIdx.x, w = t >> 6, l = t & 63, r = l & 15, c4 = l >> 4;
    constexpr int kUnit = C::kUnit, kPass = kSkPass, kRows = C::kRows, kRun = 4;
    constexpr int kCopies = 2 + ABLK;                        // operand copies of a unit
    static_assert(kRun * kSkWaves == kPass && kSkWaves >= 4 && kSkDepth <= 3, "the waits below are for at most two younger units");
    static_assert(ABLK >= 1 && ABLK <= 2, "");
    const int G = R / kGroup;
    const int j0 = blockIdx.x * 16;

    // copy offsets of this lane: block b = rows 8b..8b+7, one line per 8 lanes
    uint32_t offW[2], offX[ABLK];
    bool rowX[ABLK];                                         // this lane's row of block b exists
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int row = 8 * b + (l >> 3);
        offW[b] = (uint32_t)row * (uint32_t)R + 16 * ((l & 7) ^ ((row >> 1) & 7));
    }
#pragma unroll
    for (int b = 0; b < ABLK; ++b) {
        const int row = 8 * b + (l >> 3);
        rowX[b] = row < I;
        offX[b] = (uint32_t)min(row, I - 1) * (uint32_t)R + 16 * ((l & 7) ^ ((row >> 1) & 7));
    }
    const uint8_t* baseW = B + (size_t)j0 * R;
    // scales of a run: lanes 0 .. 31 fetch four groups of rows 0 .. 7 (clamped), the others of rows 8 .. 15 or of the block
    const int srow = l >> 2;
    const float* const gb = sb + (size_t)(j0 >> 7) * G;
    const float* const gs = (l < 32 * ABLK) ? sa + (size_t)min(srow, I - 1) * G : gb;
    const int swz = (r >> 1) & 7;
    const int frag_lo = (r >> 3) * 1024 + (r & 7) * 128 + 16 * (c4 ^ swz);
    const int frag_hi = (r >> 3) * 1024 + (r & 7) * 128 + 16 * ((4 + c4) ^ swz);

    const uint32_t ring = __builtin_amdgcn_readfirstlane(lds0 + w * C::kRing);
    const uint32_t ring_s = __builtin_amdgcn_readfirstlane(ring + kSkDepth * kUnit);
    uint8_t* const ring_p = smem + w * C::kRing;
    uint8_t* const scale_p = ring_p + kSkDepth * kUnit;
    uint8_t* const pass_p = smem + kSkWaves * C::kRing;

    // unit i of this wave is group seq(i); the wave has n_units of them.  The groups of a last, partial pass are dealt evenly.
    const int full = G / kPass, tail = G - full * kPass, run_t = (tail + kSkWaves - 1) / kSkWaves;
    auto seq = [&](int i) {
        return i < kRun * full ? (i / kRun) * kPass + w * kRun + (i % kRun) : kPass * full + w * run_t + (i - kRun * full);
    };
    const int n_units = full * kRun + max(0, min(run_t, tail - w * run_t));

    auto issue = [&](int i) {
        const int g = seq(i);
        const uint32_t u = ring + (i % kSkDepth) * kUnit;
        if (nt) {
            dma16<true>(u, baseW + (size_t)g * kGroup, offW[0]);
            dma16<true>(u + 1024, baseW + (size_t)g * kGroup, offW[1]);
        } else {
            dma16(u, baseW + (size_t)g * kGroup, offW[0]);
            dma16(u + 1024, baseW + (size_t)g * kGroup, offW[1]);
        }
        // (block b < ABLK always holds row 8 b < I, so every wave issues the same number of copies)
#pragma unroll
        for (int b = 0; b < ABLK; ++b)
            if (rowX[b]) dma16(u + 2048 + b * 1024, A + (size_t)g * kGroup, offX[b]);
        if (i % kRun == 0) {                                 // the run's scales, into the buffer that the run before last had
            const int gl = min(g + (l & 3), G - 1);
            dma4(ring_s + ((i / kRun) & 1) * C::kScales, gs + gl);
            if (ABLK == 2 && l < 4) dma4(ring_s + ((i / kRun) & 1) * C::kScales + 256, gb + gl);
        }
    };

    for (int i = 0; i < kSkDepth && i < n_units; ++i) issue(i);

    // chain owner: wave w < 4 owns the columns j0 + 4 c4 + w
    float acc = 0.0f;
    int i = 0;
    for (int g0 = 0; g0 < G; g0 += kPass) {
        const int ng = min(kPass, G - g0);
        auto unit = [&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
            if (i >= n_units) return;                // wave-uniform
            // unit i has landed once at most the younger units' copies are outstanding, and the scales behind a run's first unit
            const int younger = min(n_units, i + kSkDepth) - i - 1;
            switch (younger) {
                case 0: JET_WAIT_VMCNT(0); break;
                case 1: JET_WAIT_VMCNT(kCopies + (j + 1 >= kRun ? ABLK : 0)); break;
                default: JET_WAIT_VMCNT(2 * kCopies + (j + 2 >= kRun ? ABLK : 0)); break;
            }
            asm volatile("" ::: "memory");
            const uint8_t* u = ring_p + (i % kSkDepth) * kUnit;
            const uint8_t* us = scale_p + ((i / kRun) & 1) * C::kScales + 4 * j;
            const v8i wf = load_frag(u + frag_lo, u + frag_hi);
            const float sbv = *reinterpret_cast<const float*>(us + 128 * ABLK);
            float* dst = reinterpret_cast<float*>(pass_p + (seq(i) - g0) * C::kGroupBytes);
            const v8i xf = load_frag(u + 2048 + frag_lo, u + 2048 + frag_hi);
            const float s = *reinterpret_cast<const float*>(us + 16 * (r & (8 * ABLK - 1))) * sbv;
            const v4f p = group_product(wf, xf);
            if (kRows == 16 || r < 8) {
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(4 * e + c4) * kRows + r] = p[e];
                dst[(16 + c4) * kRows + r] = s;
            }
            asm volatile("" ::: "memory");
            if (i + kSkDepth < n_units) issue(i + kSkDepth);
            ++i;
        };
        unit(std::integral_constant<int, 0>{});
        unit(std::integral_constant<int, 1>{});
        unit(std::integral_constant<int, 2>{});
        unit(std::integral_constant<int, 3>{});
        __syncthreads();
        if (w < 4) {                                     // wave-uniform
            const float* src_p = reinterpret_cast<const float*>(pass_p) + (4 * w + c4) * kRows + (r & (kRows - 1));
            const float* src_s = reinterpret_cast<const float*>(pass_p) + (16 + c4) * kRows + (r & (kRows - 1));
            if (ng == kPass) {
                // all LDS reads of the pass first, then the ordered chain: a loop of read, read, fma
                // pays the LDS latency once per group (1.6 us per pass of 32 groups)
                float pv[kPass], sv[kPass];
#pragma unroll
                for (int g = 0; g < kPass; ++g) {
                    pv[g] = src_p[g * (C::kGroupBytes / 4)];
                    sv[g] = src_s[g * (C::kGroupBytes / 4)];
                }
#pragma unroll
                for (int g = 0; g < kPass; ++g) acc = chain(pv[g], sv[g], acc);
            } else {
                for (int g = 0; g < ng; ++g) acc = chain(src_p[g * (C::kGroupBytes / 4)], src_s[g * (C::kGroupBytes / 4)], acc);
            }
        }
        __syncthreads();
    }
    if (w < 4 && r < I) out[(size_t)r * J + j0 + 4 * c4 + w] = (uint16_t)bf16_rne(acc);
}

// ------------------------------------------------------------------------
// Panel kernel (block scales only): batches of up to 1024 rows, and larger ones against narrow matrices, where
// jet_plan.h prefers it.  One workgroup per CU owns a BM x BN output tile and walks the
// whole reduction, a step of one, two or four groups at a time; WR x WC waves compute, kCopy waves copy the operands and
// one the scales.
// What bounds it: a CU can have about 320 cache lines on their way and gets them back in order, so an
// activation line (an L2 hit) waits behind the weight lines (HBM misses) in front of it.  A tile takes about
// (BM + BN) * G * 2.4 ns, whatever its lines hit (measured from 48 to 240 lines per group), plus 3-4 us of launch, ring
// fill and output.  So lines decide the tile (jet_plan.h), and a wide matrix gets wide tiles: the
// activations of a group pass once per 112 columns and not once per 32.
// Ring of S stages, per group [W: BN rows x 128][A: BM rows x 128] in the swizzled fragment layout of the tile
// kernel; scales travel in chunks of 16 groups, [row][16] with the group xor (row >> 2) & 3 (conflict-free), two buffers.
// The computing waves fetch the fragments of the next group into registers while they compute one; before the last group
// of step p, when all of the step is in registers, the barrier: the copying waves have waited until step p+1 has
// landed and now refill the slot of step p with step p+S.  As many groups per step as the LDS takes with three stages:
// the copies of a row then fetch 256 or 512 bytes at a time (all CUs walk the same 128-byte column of rows 4 KB apart), and
// there are fewer barriers: 2-8 % over a step of one or two groups.  The activations of a step go out in front of its weights:
// hits in front of misses do not wait for them (28 shapes of 32 to 256 rows from HBM 1.5 % faster than behind them, us:
// 4096x4096 32 rows 7.35 -> 7.07, 128 rows 9.29 -> 8.85; 4096x14336 128 rows 24.4 -> 23.6; 5120x27648 256 rows 75.9 -> 74.3;
// block by block in turn as slow as the weights first).  336 shapes of 17 to 600 rows and 16 matrices, activations in the caches:
// 1.7 % faster on average where the weights are read past the caches (118 shapes, at worst 17x4096x4096 6.9 -> 7.2 and 48 to 90 rows
// of 28672x4096 2 % slower), 1.7 % through them beside a partly filled row block (161, at worst 1.2 % slower), 0.5 % below 16 MB (57);
// activations from HBM as well 2.4, 0.5 and -0.2 %, at worst 150x4096x28672 58.3 -> 59.9.  The copying loop is
// straight-line (a compare chain for the wait and a branch per copy cost 0.3 us per step), and the fetch stays in front
// of the MFMAs by scheduling barriers.  Every output element takes the chain of the other kernels.
// From HBM, against the strip kernel of 64x32 and 32x32 tiles and the 128x128 tiles before it (us): 4096x14336 77 rows
// 27.8 -> 20.9, 128 rows 29.5 -> 24.8, 256 rows 54.9 -> 35.8; 28672x4096 32 rows 32.3 -> 27.3, 64 rows 45.6 -> 29.2; 6144x4096
// 128 rows 22.2 -> 13.4; 5120x27648 64 rows 55.7 -> 44.0, 256 rows 146 -> 76; 55296x5120 64 rows 100 -> 58.  The copying side alone takes 90 % of
// that, the computing side alone 55-85 %; the weights without the activations 16.7 of 29 us (4096x14336, 128 rows).
// Measured and left out: workgroups on idle CUs that pull the weights into the L2 ahead (32-row tiles of 4096x14336
// 22.4 -> 18.1 us, elsewhere within 10 % either way), a wave that touches the XCD's weight lines a chunk ahead (its
// burst holds up the barrier: 30 % slower), the workgroups of an XCD touching its activation lines once at the start (dealt
// among those that share a row block, 2-5 % slower than without, 139 shapes of one to five row blocks; the first copies wait).
// ------------------------------------------------------------------------
template <int TM_, int TN_, int WR_, int WC_, int S_, int GP_ = 1>
struct PanelCfg {
    static constexpr int TM = TM_, TN = TN_, WR = WR_, WC = WC_, S = S_, GP = GP_;
    static constexpr int BM = 16 * TM * WR, BN = 16 * TN * WC;
    static constexpr int kWBlocks = BN / 8, kABlocks = BM / 8;            // 1 KB copies of a group
    static constexpr int kCopy = (kWBlocks % 4 == 0 && kABlocks % 4 == 0 && WR * WC <= 3) ? 4 : 2;
    static constexpr int kCompute = WR * WC, kThreads = 64 * (kCompute + kCopy + 1);
    static constexpr int kWPer = kWBlocks / kCopy, kAPer = kABlocks / kCopy, kPer = GP * (kWPer + kAPer);
    static constexpr int kGroupBytes = (BM + BN) * 128, kStage = GP * kGroupBytes;
    static constexpr int kChunk = 16, kSaBuf = BM * kChunk * 4, kSbBuf = 256;
    static constexpr int kSaOff = S * kStage, kSbOff = kSaOff + 2 * kSaBuf;
    static constexpr int kLds = kSbOff + 2 * kSbBuf;
    static_assert(kWBlocks % kCopy == 0 && kABlocks % kCopy == 0, "");
    static_assert(S >= 3 && (S - 1) * kPer < 64 && BN <= 256 && kLds <= 160 * 1024 && kChunk % GP == 0, "");
};

// wait until at most n steps' copies (kCnt each) of this wave are outstanding
template <int kCnt, int kMax>
__device__ __forceinline__ void wait_steps(int n) {
    if (n >= kMax) {
        JET_WAIT_VMCNT(kMax * kCnt);
    } else if constexpr (kMax > 0) {
        wait_steps<kCnt, kMax - 1>(n);
    }
}
__device__ __forceinline__ void step_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <class C>
__global__ __launch_bounds__(C::kThreads) void gemm_panel_kernel(const uint8_t* __restrict__ A,
                                                                  const float* __restrict__ sa,
                                                                  const uint8_t* __restrict__ B,
                                                                  const float* __restrict__ sb,
                                                                  uint16_t* __restrict__ out, int I, int J, int ldo, int R,
                                                                  int row_blocks, bool nt) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, r = l & 15, c4 = l >> 4;
    const int G = R / kGroup, P = (G + C::GP - 1) / C::GP;
    // row blocks that share a weight panel are neighbours on one XCD, so the panel leaves HBM once
    const int id = xcd_contiguous_id(blockIdx.x, gridDim.x);
    const int rb = id % row_blocks, panel = id / row_blocks;
    const int i0 = rb * C::BM, j0 = panel * C::BN;

    if (w >= C::kCompute + C::kCopy) {
        // ---------------- scale wave: chunks of 16 groups, two buffers ----------------
        auto copy_chunk = [&](int c) {
            const uint32_t sa_dst = lds0 + C::kSaOff + (c & 1) * C::kSaBuf;
            for (int rq = 0; rq < C::BM / 4; ++rq) {     // rows 4 rq .. 4 rq + 3
                const int row = min(i0 + 4 * rq + (l >> 4), I - 1), g = min(C::kChunk * c + ((l & 15) ^ (rq & 3)), G - 1);
                dma4(sa_dst + rq * 256, sa + (size_t)row * G + g);
            }
            const int blk = min((j0 >> 7) + (l >> 4), (J >> 7) - 1), g = min(C::kChunk * c + (l & 15), G - 1);
            dma4(lds0 + C::kSbOff + (c & 1) * C::kSbBuf, sb + (size_t)blk * G + g);
        };
        constexpr int kSteps = C::kChunk / C::GP;        // steps of a chunk
        copy_chunk(0);
        JET_WAIT_VMCNT(0);
        step_barrier();
        for (int p = 0, k = 0, c = 0; p < P; ++p) {
            if (k == kSteps - 1) JET_WAIT_VMCNT(0);      // chunk c + 1: its first fetch follows this barrier
            step_barrier();
            if (k == 0 && (c + 1) * C::kChunk < G) copy_chunk(c + 1);   // nobody reads chunk c - 1 any more
            if (++k == kSteps) { k = 0; ++c; }
        }
        JET_WAIT_VMCNT(0);
        return;
    }
    if (w >= C::kCompute) {
        // ---------------- copying waves: blocks cw, cw + kCopy, ... of every group ----------------
        const int cw = w - C::kCompute;
        const uint8_t* baseW = static_cast<const uint8_t*>(uniform_ptr(B + (size_t)j0 * R));
        const uint8_t* baseA = static_cast<const uint8_t*>(uniform_ptr(A + (size_t)i0 * R));
        const uint32_t lane_chunk = (16 * ((l & 7) ^ (l >> 4))) ^ ((cw & 1) * 64);
        uint32_t offW[C::kWPer], offA[C::kAPer];         // rows and columns past the end repeat the last one (never stored)
#pragma unroll
        for (int i = 0; i < C::kWPer; ++i)
            offW[i] = (uint32_t)(min(j0 + 8 * (cw + C::kCopy * i) + (l >> 3), J - 1) - j0) * (uint32_t)R + lane_chunk;
#pragma unroll
        for (int i = 0; i < C::kAPer; ++i)
            offA[i] = (uint32_t)(min(i0 + 8 * (cw + C::kCopy * i) + (l >> 3), I - 1) - i0) * (uint32_t)R + lane_chunk;
        const uint32_t lds_c = __builtin_amdgcn_readfirstlane(lds0 + cw * 1024);
        uint32_t st = lds_c;
        auto copy_steps = [&](auto nt_tag) {             // straight-line for either policy of the weights
            constexpr bool kNt = decltype(nt_tag)::value;
            auto issue = [&](int q) {
                size_t kb[C::GP];                        // past the end: the last group again
#pragma unroll
                for (int h = 0; h < C::GP; ++h) kb[h] = (size_t)min(C::GP * q + h, G - 1) * kGroup;
                // the activations first (the panel's comment), the groups of a row next to each other
#pragma unroll
                for (int i = 0; i < C::kAPer; ++i)
#pragma unroll
                    for (int h = 0; h < C::GP; ++h)
                        dma16(st + h * C::kGroupBytes + C::BN * 128 + i * (C::kCopy * 1024), baseA + kb[h], offA[i]);
#pragma unroll
                for (int i = 0; i < C::kWPer; ++i)
#pragma unroll
                    for (int h = 0; h < C::GP; ++h)
                        dma16<kNt>(st + h * C::kGroupBytes + i * (C::kCopy * 1024), baseW + kb[h], offW[i]);
                st = (st == lds_c + (C::S - 1) * C::kStage) ? lds_c : st + C::kStage;
            };
            for (int q = 0; q < C::S && q < P; ++q) issue(q);
            wait_steps<C::kPer, C::S - 1>(min(P, C::S) - 1); // step 0
            step_barrier();
            int p = 0;
            for (; p + C::S < P; ++p) {
                JET_WAIT_VMCNT((C::S - 2) * C::kPer);        // step p + 1; younger: p + 2 .. p + S - 1
                step_barrier();
                issue(p + C::S);
            }
            for (; p < P; ++p) {
                wait_steps<C::kPer, C::S - 1>(max(P - p - 2, 0));
                step_barrier();
            }
        };
        if (nt) copy_steps(std::true_type{});
        else copy_steps(std::false_type{});
        JET_WAIT_VMCNT(0);   // nothing may be in flight towards the LDS when it is released
        return;
    }

    // ---------------- computing waves ----------------
    const int wr = w / C::WC, wc = w % C::WC;
    const int swz = (r >> 1) & 7;
    const int frag_lo = (r >> 3) * 1024 + (r & 7) * 128 + 16 * (c4 ^ swz);
    const int frag_hi = (r >> 3) * 1024 + (r & 7) * 128 + 16 * ((4 + c4) ^ swz);
    const uint8_t* const pw0 = smem + wc * C::TN * 2048;
    const uint8_t* const pa0 = smem + C::BN * 128 + wr * C::TM * 2048;
    const uint8_t* const ps0 = smem + C::kSaOff + (wr * C::TM * 16 + r) * 64;
    const int sa_xor = ((r >> 2) & 3) * 4;
    int sb_off[C::TN];                                   // block of a column tile in the chunk of block scales
#pragma unroll
    for (int n = 0; n < C::TN; ++n) sb_off[n] = (((j0 + 16 * (wc * C::TN + n)) >> 7) - (j0 >> 7)) * 64;
    struct Operands {
        v8i wf[C::TN], xf[C::TM];
        float sa[C::TM], sb[C::TN];
    };
    auto fetch = [&](int g, int base, Operands& o) {     // group g, at LDS offset base
        const int buf = (g / C::kChunk) & 1, k4 = (g % C::kChunk) * 4;
        const uint8_t* pw = pw0 + base;
        const uint8_t* pa = pa0 + base;
        const uint8_t* ps = ps0 + buf * C::kSaBuf + (k4 ^ sa_xor);
        const uint8_t* pb = smem + C::kSbOff + buf * C::kSbBuf + k4;
#pragma unroll
        for (int m = 0; m < C::TM; ++m) {
            o.xf[m] = load_frag(pa + m * 2048 + frag_lo, pa + m * 2048 + frag_hi);
            o.sa[m] = *reinterpret_cast<const float*>(ps + m * 1024);
        }
#pragma unroll
        for (int n = 0; n < C::TN; ++n) {
            o.wf[n] = load_frag(pw + n * 2048 + frag_lo, pw + n * 2048 + frag_hi);
            o.sb[n] = *reinterpret_cast<const float*>(pb + sb_off[n]);
        }
    };
    v4f acc[C::TM][C::TN];
#pragma unroll
    for (int m = 0; m < C::TM; ++m)
#pragma unroll
        for (int n = 0; n < C::TN; ++n) acc[m][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    auto compute = [&](const Operands& o) {
        constexpr int kTiles = C::TM * C::TN, kLag = kTiles < 2 ? kTiles : 2;
        v4f pr[3];
#pragma unroll
        for (int u = 0; u < kTiles + kLag; ++u) {
            if (u < kTiles) pr[u % 3] = group_product(o.wf[u % C::TN], o.xf[u / C::TN]);
            if (u >= kLag) {
                const int v = u - kLag, m = v / C::TN, n = v % C::TN;
                const float s = o.sa[m] * o.sb[n];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[m][n][e] = chain(pr[v % 3][e], s, acc[m][n][e]);
            }
        }
    };
    step_barrier();                                      // step 0 has landed
    Operands even, odd;
    fetch(0, 0, even);
    int stage = 0;
    // one group: `cur` holds its fragments, the next group's go to `nxt`.  Before the last group of a step the barrier:
    // the step's fragments are all in registers, so its slot may be overwritten, and the next step has landed.
    auto group = [&](int g, int h, const Operands& cur, Operands& nxt) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0)
        if (h == C::GP - 1) {
            step_barrier();
            stage = (stage == (C::S - 1) * C::kStage) ? 0 : stage + C::kStage;
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch(g + 1, stage + (h == C::GP - 1 ? 0 : (h + 1) * C::kGroupBytes), nxt);   // (after the last: whatever is there, not used)
        __builtin_amdgcn_sched_barrier(0);
        if (g < G) compute(cur);                         // a last step may hold fewer groups
    };
    static_assert(C::GP == 1 || C::GP % 2 == 0, "the two operand buffers alternate");
    int p = 0;
    if constexpr (C::GP == 1) {
        for (; p + 1 < P; p += 2) {
            group(p, 0, even, odd);
            group(p + 1, 0, odd, even);
        }
        if (p < P) group(p, 0, even, odd);
    } else {
        for (; p < P; ++p) {
#pragma unroll
            for (int h = 0; h < C::GP; h += 2) {
                group(C::GP * p + h, h, even, odd);
                group(C::GP * p + h + 1, h + 1, odd, even);
            }
        }
    }

#pragma unroll
    for (int m = 0; m < C::TM; ++m) {
        const int i = i0 + (wr * C::TM + m) * 16 + r;
#pragma unroll
        for (int n = 0; n < C::TN; ++n) {
            const int j = j0 + (wc * C::TN + n) * 16 + 4 * c4;
            uint2 o;
            o.x = bf16_pack2(acc[m][n][0], acc[m][n][1]);
            o.y = bf16_pack2(acc[m][n][2], acc[m][n][3]);
            if (i < I && j < J) *reinterpret_cast<uint2*>(out + (size_t)i * ldo + j) = o;
        }
    }
}

// ----------------------------------------------------------------- launch --

template <typename K>
static hipError_t allow_lds(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// big tile: 256x256, 8 waves of 128x64;  wide tile: 256x128, 8 waves of 64x64, three stages;  small tile: 128x128, 4 waves of 64x64
#define JET_BIG 2, 4, 8, 4
#define JET_WIDE 4, 2, 4, 4, 3
#define JET_SMALL 2, 2, 4, 4
#define JET_SMALL_DEEP 2, 2, 4, 4, 4   /* four stages, one workgroup per CU: copies three steps ahead */
#define JET_HALF 4, 1, 2, 4, 4         /* 128x64 tile, 4 waves of 32x64, four stages */

// compute units of the current device (256 on MI355X), asked once per process
static int compute_units() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
            v = 256;
        return v;
    }();
    return n;
}

template <class C>
static hipError_t launch_panel(const uint8_t* A, const float* sa, const uint8_t* B, const float* sb, uint16_t* o, long I,
                               long J, long R, long ldo, bool nt, hipStream_t st) {
    const int rbs = (int)((I + C::BM - 1) / C::BM);
    const long panels = (J + C::BN - 1) / C::BN;
    hipLaunchKernelGGL((gemm_panel_kernel<C>), dim3((unsigned)(rbs * panels)), dim3(C::kThreads), C::kLds, st, A, sa, B,
                       sb, o, (int)I, (int)J, (int)ldo, (int)R, rbs, nt);
    return hipGetLastError();
}

using PanelLaunch = hipError_t (*)(const uint8_t*, const float*, const uint8_t*, const float*, uint16_t*, long, long, long,
                                   long, bool, hipStream_t);
#define JET_PANEL_LAUNCH(TM, TN, WR, WC, S, GP, GROUP, ROUND) launch_panel<PanelCfg<TM, TN, WR, WC, S, GP>>,
static const PanelLaunch kPanelLaunches[] = {JET_PANELS(JET_PANEL_LAUNCH)};
#undef JET_PANEL_LAUNCH
static_assert(std::size(kPanelLaunches) == kNumPanels, "the panels come first in kGemmTiles");

template <GemmKernel KERNEL, int SB_MODE, int... Cfg>
static hipError_t launch_tiles(const uint8_t* A, const float* sa, const uint8_t* B, const float* sb, uint16_t* o, long I,
                               long J, long R, long ldo, hipStream_t st) {
    using C = TileCfg<SB_MODE, Cfg...>;
    static_assert(C::kOccupancy == resident_per_cu(KERNEL), "the plan's rounds");
    const long ti = (I + C::BM - 1) / C::BM, tj = J / C::BN;
    const long wgs = std::min<long>(ti * tj, (long)compute_units() * C::kOccupancy);
    hipLaunchKernelGGL((gemm_tile_kernel<SB_MODE, Cfg...>), dim3((unsigned)wgs), dim3(C::kThreads), C::kLdsBytes, st, A,
                       sa, B, sb, o, (int)I, (int)ldo, (int)R, (int)ti, (int)tj, reciprocal((unsigned)(8 * tj)),
                       reciprocal((unsigned)std::max<long>(ti % 8, 1)));
    return hipGetLastError();
}

// decode of up to 16 rows: a workgroup per 16-column strip
static hipError_t launch_strips(const uint8_t* A, const float* sa, const uint8_t* B, const float* sb, uint16_t* o, long I,
                                long J, long R, int depth, bool nt, hipStream_t st) {
    const unsigned strips = (unsigned)(J / 16);
#define JET_SKINNY_AB(D, W, AB)                                                                             \
    hipLaunchKernelGGL((gemm_skinny_kernel<D, W, AB>), dim3(strips), dim3(64 * W), (SkinnyCfg<D, W, AB>::kLds), st, A, \
                       sa, B, sb, o, (int)I, (int)J, (int)R, nt)
    // copy only the 8-row activation blocks that hold a row of the batch
#define JET_SKINNY(D, W)                       \
    do {                                       \
        if (I <= 8) JET_SKINNY_AB(D, W, 1);    \
        else JET_SKINNY_AB(D, W, 2);           \
    } while (0)
    if (depth == 3) JET_SKINNY(3, 8);                           // a workgroup per CU
    else if (depth == 1) JET_SKINNY(1, 8);                      // two (16 waves) per CU
    else if (I <= 8) JET_SKINNY_AB(2, 8, 1);                    // two, more than one round of them
    else return hipErrorInvalidValue;
#undef JET_SKINNY
#undef JET_SKINNY_AB
    return hipGetLastError();
}

// out has row pitch ldo (>= J): a split plan runs the kernels on row or column ranges of a larger problem
template <int SB_MODE>
static hipError_t launch_planned(const uint8_t* A, const float* sa, const uint8_t* B, const float* sb, uint16_t* o, long I,
                                 long J, long R, long ldo, hipStream_t st, bool whole = true) {
    const long G = R / kGroup;
    const GemmPlan p = plan_gemm(SB_MODE == kSbRow, I, J, G, compute_units(), whole);
    switch (p.kernel) {
        case kStrips:
            if constexpr (SB_MODE == kSbBlock) return launch_strips(A, sa, B, sb, o, I, J, R, p.depth, p.nt, st);
            break;
        case kPanel:
            if constexpr (SB_MODE == kSbBlock) return kPanelLaunches[p.panel](A, sa, B, sb, o, I, J, R, ldo, p.nt, st);
            break;
        case kTileWide:
            if constexpr (SB_MODE == kSbBlock) return launch_tiles<kTileWide, kSbBlock, JET_WIDE>(A, sa, B, sb, o, I, J, R, ldo, st);
            break;
        case kTileHalf:
            if constexpr (SB_MODE == kSbBlock) return launch_tiles<kTileHalf, kSbBlock, JET_HALF>(A, sa, B, sb, o, I, J, R, ldo, st);
            break;
        case kTileBig: return launch_tiles<kTileBig, SB_MODE, JET_BIG>(A, sa, B, sb, o, I, J, R, ldo, st);
        case kTileSmallDeep: return launch_tiles<kTileSmallDeep, SB_MODE, JET_SMALL_DEEP>(A, sa, B, sb, o, I, J, R, ldo, st);
        case kTileSmall: return launch_tiles<kTileSmall, SB_MODE, JET_SMALL>(A, sa, B, sb, o, I, J, R, ldo, st);
        case kSplitRows: {
            const hipError_t e = launch_planned<SB_MODE>(A, sa, B, sb, o, p.split, J, R, ldo, st, false);
            if (e != hipSuccess) return e;
            return launch_planned<SB_MODE>(A + p.split * R, sa + p.split * G, B, sb, o + p.split * ldo, I - p.split, J, R, ldo, st,
                                           false);
        }
        case kSplitCols: {
            const hipError_t e = launch_planned<SB_MODE>(A, sa, B, sb, o, I, p.split, R, ldo, st, false);
            if (e != hipSuccess) return e;
            const float* sb_tail = sb + (SB_MODE == kSbBlock ? (p.split / kGroup) * G : p.split * G);
            return launch_planned<SB_MODE>(A, sa, B + p.split * R, sb_tail, o + p.split, I, J - p.split, R, ldo, st, false);
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(const uint8_t* A, const float* sa, const uint8_t* B, const float* sb,
                       int sb_mode, void* out, long I, long J, long R, hipStream_t st) {
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        hipError_t e = hipSuccess;
        auto allow_tiles = [&](auto kernel, int bytes) {
            if (e == hipSuccess) e = allow_lds(kernel, bytes);
        };
#define JET_TILE_ATTR(MODE, ...) allow_tiles(gemm_tile_kernel<MODE, __VA_ARGS__>, TileCfg<MODE, __VA_ARGS__>::kLdsBytes)
        JET_TILE_ATTR(kSbBlock, JET_BIG);
        JET_TILE_ATTR(kSbRow, JET_BIG);
        JET_TILE_ATTR(kSbBlock, JET_WIDE);
        JET_TILE_ATTR(kSbBlock, JET_HALF);
        JET_TILE_ATTR(kSbBlock, JET_SMALL);
        JET_TILE_ATTR(kSbRow, JET_SMALL);
        JET_TILE_ATTR(kSbBlock, JET_SMALL_DEEP);
        JET_TILE_ATTR(kSbRow, JET_SMALL_DEEP);
#undef JET_TILE_ATTR
#define JET_SK_ATTR(D, W, AB) \
    if (e == hipSuccess) e = allow_lds(gemm_skinny_kernel<D, W, AB>, SkinnyCfg<D, W, AB>::kLds)
        JET_SK_ATTR(3, 8, 1); JET_SK_ATTR(3, 8, 2);
        JET_SK_ATTR(1, 8, 1); JET_SK_ATTR(1, 8, 2); JET_SK_ATTR(2, 8, 1);
#undef JET_SK_ATTR
#define JET_PANEL_ATTR(TM, TN, WR, WC, S, GP, GROUP, ROUND) \
    if (e == hipSuccess) e = allow_lds(gemm_panel_kernel<PanelCfg<TM, TN, WR, WC, S, GP>>, PanelCfg<TM, TN, WR, WC, S, GP>::kLds);
        JET_PANELS(JET_PANEL_ATTR)
#undef JET_PANEL_ATTR
        attr_err = e;
    });
    if (attr_err != hipSuccess) return attr_err;

    uint16_t* o = static_cast<uint16_t*>(out);
    if (sb_mode == kSbBlock) return launch_planned<kSbBlock>(A, sa, B, sb, o, I, J, R, J, st);
    return launch_planned<kSbRow>(A, sa, B, sb, o, I, J, R, J, st);
}

}  // namespace jet
