// Fused amax / scale / cast quantizers (Jet-RL Sec. 2.1 formula at the
// granularities of Sec. 4.2).  All of them are HBM-bound streaming kernels:
// every input byte is read once with 16-byte loads, every output byte written
// once, reductions stay in registers (DPP) or LDS.
#include "jet_internal.h"
#include "jet_numerics.h"
#include "jet_tile_quant.h"

namespace jet {

// ------------------------------------------------------------------------
// Row quantizer: 1x128 groups along the contiguous axis.  A team of 8 lanes
// owns one group; a lane owns 16 consecutive elements (32 B of bf16 in, 16 B
// of codes out).  Works for any M (decode shapes included).
// ------------------------------------------------------------------------
template <int SRC>
__global__ __launch_bounds__(256) void quant_row_kernel(const void* __restrict__ x,
                                                        const float* __restrict__ xs,
                                                        uint8_t* __restrict__ q,
                                                        float* __restrict__ s, long n_groups) {
    const long n_teams = (long)gridDim.x * 32;
    const int l8 = threadIdx.x & 7;
    for (long g = ((long)blockIdx.x * 256 + threadIdx.x) >> 3; g < n_groups; g += n_teams) {
        float v[16];
        if (SRC == JET_SRC_BF16) {
            const uint4* p = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + g * kGroup + l8 * 16);
            uint4 u0 = p[0], u1 = p[1];
            const uint32_t w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[2 * i] = bf16_lo(w[i]);
                v[2 * i + 1] = bf16_hi(w[i]);
            }
        } else {
            const uint4 u = *reinterpret_cast<const uint4*>(static_cast<const uint8_t*>(x) + g * kGroup + l8 * 16);
            const float sc = xs[g];
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float a, b, c, d;
                e4m3_unpack4(w[i], a, b, c, d);
                v[4 * i] = a * sc;
                v[4 * i + 1] = b * sc;
                v[4 * i + 2] = c * sc;
                v[4 * i + 3] = d * sc;
            }
        }
        float am = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) am = fmaxf(am, fabsf(v[i]));
        am = team8_max(am);
        const GroupScale gs = make_scale(am);
        uint32_t o[4];
        encode<SRC == JET_SRC_BF16 ? kBf16Values : kFloatValues>(v, gs, o);
        *reinterpret_cast<uint4*>(q + g * kGroup + l8 * 16) = uint4{o[0], o[1], o[2], o[3]};
        if (l8 == 0) s[g] = gs.S;
    }
}

// ------------------------------------------------------------------------
// Tile quantizer: one workgroup per 128x128 tile of the source.
//   ROW  : 1x128 groups along the contiguous axis   -> q_row, s_row
//   COL  : 128x1 groups along the row axis, outputs transposed -> q_colT, s_colT
//   BLOCK: one scale for the whole tile (weights); q_row/s_row are the plain
//          outputs, q_colT/s_colT the optional transposed copy (COL says whether
//          it is wanted).
// Thread (rr = t>>4, cc = t&15) holds rows 8rr..8rr+7, columns 8cc..8cc+7 of the
// tile as binary32, so that codes pack along either axis without shuffles; the
// transposed bytes go through LDS once so that global stores are 16 B wide.
// Two bytes in and at most two out per element, but about ten vector instructions: a scale (two IEEE
// divisions, 25 instructions) is therefore formed once per group and not by each of the threads that hold it.
// Before that, with a branch per element and conflicts on the maxima in LDS, the kernel was bound by its
// instructions.  [16384, 4096]: row + column 59 -> 49.5 us, column from FP8 30 -> 25; [128, 4096]: 8.9 -> 5.0 and
// 5.5 -> 4.3; a weight with its transposed copy [128, 4096] 5.2 -> 3.5, 14 matrices of two 8B layers 399 -> 377.
// The source is read past the memory-side cache (gradients, FP8-saved activations and master weights are not read
// again soon), so that what is written stays in it: row + column [16384, 1024] 17.4 -> 15.0 us, column from FP8 [16384, 14336]
// 132 -> 123, a weight [4096, 4096] 11.9 -> 10.6, with its transposed copy 15.0 -> 13.5.  Stores past it as well would
// gain 3-8 % more here and cost the GEMM that reads the codes next as much or more (weight [14336, 4096] and the FProp of 32
// rows behind it 51 -> 55 us); the row quantizer, whose source the operator before has just written, gains nothing.  A source that
// a copy has just written (copy and quantizer together): 3 to 8 % faster from 8192x14336 on, 4096x4096 and 16384x1024 weights
// 20.9 -> 21.8 us.  With an operator behind that reads the source again: 0.94 to 1.08, the worst 4096x14336 with
// its transposed copy, 119 -> 128 us.
// ------------------------------------------------------------------------

template <int SRC, bool ROW, bool COL, bool BLOCK>
__global__ __launch_bounds__(256) void quant_tile_kernel(const void* __restrict__ x,
                                                         const float* __restrict__ xs, long M, long K,
                                                         uint8_t* __restrict__ q_row,
                                                         float* __restrict__ s_row,
                                                         uint8_t* __restrict__ q_colT,
                                                         float* __restrict__ s_colT) {
    constexpr ValueKind kKind = SRC == JET_SRC_BF16 ? kBf16Values : kFloatValues;
    __shared__ __attribute__((aligned(16))) TileLds L;

    const int t = threadIdx.x, rr = t >> 4, cc = t & 15, w = t >> 6;
    const long m0 = (long)blockIdx.y * 128, k0 = (long)blockIdx.x * 128;
    const long GK = K / kGroup, GM = M / kGroup;

    float v[8][8];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const long row = m0 + 8 * rr + p;
        if (SRC == JET_SRC_BF16) {
            const uint4 u = load16_nt(static_cast<const uint16_t*>(x) + row * K + k0 + 8 * cc);
            v[p][0] = bf16_lo(u.x); v[p][1] = bf16_hi(u.x);
            v[p][2] = bf16_lo(u.y); v[p][3] = bf16_hi(u.y);
            v[p][4] = bf16_lo(u.z); v[p][5] = bf16_hi(u.z);
            v[p][6] = bf16_lo(u.w); v[p][7] = bf16_hi(u.w);
        } else {
            const uint2 u = load8_nt(static_cast<const uint8_t*>(x) + row * K + k0 + 8 * cc);
            const float sc = xs[row * GK + blockIdx.x];
            e4m3_unpack4(u.x, v[p][0], v[p][1], v[p][2], v[p][3]);
            e4m3_unpack4(u.y, v[p][4], v[p][5], v[p][6], v[p][7]);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[p][j] *= sc;
        }
    }

    if (BLOCK) {
        // one amax for the tile: lanes -> 16-lane rows -> wave -> workgroup
        float am = 0.0f;
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int j = 0; j < 8; ++j) am = fmaxf(am, fabsf(v[p][j]));
        am = team16_max(am);
        am = fmaxf(am, __shfl_xor(am, 16));
        am = fmaxf(am, __shfl_xor(am, 32));
        if ((t & 63) == 0) L.red[w] = am;
        __syncthreads();
        am = fmaxf(fmaxf(L.red[0], L.red[1]), fmaxf(L.red[2], L.red[3]));
        const GroupScale gs = make_scale(am);
        if (t == 0) {
            s_row[(long)blockIdx.y * GK + blockIdx.x] = gs.S;
            if (COL) s_colT[(long)blockIdx.x * GM + blockIdx.y] = gs.S;
        }
        uint32_t o[8][2];
        if (gs.plain) {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                o[p][0] = codes4<kKind>(v[p][0], v[p][1], v[p][2], v[p][3], gs.S, gs.r);
                o[p][1] = codes4<kKind>(v[p][4], v[p][5], v[p][6], v[p][7], gs.S, gs.r);
            }
        } else {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                o[p][0] = codes4_any(v[p][0], v[p][1], v[p][2], v[p][3], gs.S);
                o[p][1] = codes4_any(v[p][4], v[p][5], v[p][6], v[p][7], gs.S);
            }
        }
#pragma unroll
        for (int p = 0; p < 8; ++p)
            *reinterpret_cast<uint2*>(q_row + (m0 + 8 * rr + p) * K + k0 + 8 * cc) = uint2{o[p][0], o[p][1]};
        if (COL) {
            // the same codes along the other axis: 4x4 byte transposes
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t up[4], dn[4];
                transpose4(o[0][h], o[1][h], o[2][h], o[3][h], up);
                transpose4(o[4][h], o[5][h], o[6][h], o[7][h], dn);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<uint2*>(&L.T[t_addr(8 * cc + 4 * h + j, rr >> 1) + 8 * (rr & 1)]) = uint2{up[j], dn[j]};
            }
        }
        if (COL) store_transposed(L, m0, k0, M, q_colT);
    } else {
        quantize_tile<kKind, ROW, COL>(v, L, m0, k0, M, K, q_row, s_row, q_colT, s_colT);
    }
}

// ----------------------------------------------------------------- launch --

template <int SRC>
static hipError_t launch_row(const void* x, const float* xs, long M, long K, uint8_t* q, float* s,
                             hipStream_t st) {
    const long n_groups = M * (K / kGroup);
    long blocks = (n_groups + 31) / 32;
    const long cap = 256L * 32;  // a few waves of workgroups per CU, grid-stride beyond that
    if (blocks > cap) blocks = cap;
    hipLaunchKernelGGL((quant_row_kernel<SRC>), dim3((unsigned)blocks), dim3(256), 0, st, x, xs, q, s, n_groups);
    return hipGetLastError();
}

template <int SRC, bool ROW, bool COL, bool BLOCK>
static hipError_t launch_tile(const void* x, const float* xs, long M, long K, uint8_t* q_row,
                              float* s_row, uint8_t* q_colT, float* s_colT, hipStream_t st) {
    dim3 grid((unsigned)(K / 128), (unsigned)(M / 128));
    hipLaunchKernelGGL((quant_tile_kernel<SRC, ROW, COL, BLOCK>), grid, dim3(256), 0, st, x, xs, M, K,
                       q_row, s_row, q_colT, s_colT);
    return hipGetLastError();
}

hipError_t launch_quant_act(const void* x, const float* xs, int src, long M, long K, uint8_t* q_row,
                            float* s_row, uint8_t* q_colT, float* s_colT, hipStream_t st) {
    const bool row = q_row != nullptr, col = q_colT != nullptr;
    if (src == JET_SRC_BF16) {
        if (row && col) return launch_tile<JET_SRC_BF16, true, true, false>(x, xs, M, K, q_row, s_row, q_colT, s_colT, st);
        if (col) return launch_tile<JET_SRC_BF16, false, true, false>(x, xs, M, K, q_row, s_row, q_colT, s_colT, st);
        return launch_row<JET_SRC_BF16>(x, xs, M, K, q_row, s_row, st);
    }
    if (row && col) return launch_tile<JET_SRC_FP8_ROW, true, true, false>(x, xs, M, K, q_row, s_row, q_colT, s_colT, st);
    if (col) return launch_tile<JET_SRC_FP8_ROW, false, true, false>(x, xs, M, K, q_row, s_row, q_colT, s_colT, st);
    return launch_row<JET_SRC_FP8_ROW>(x, xs, M, K, q_row, s_row, st);
}

hipError_t launch_quant_weight(const void* w, long N, long K, uint8_t* q, float* s, uint8_t* qT,
                               float* sT, hipStream_t st) {
    if (qT) return launch_tile<JET_SRC_BF16, true, true, true>(w, nullptr, N, K, q, s, qT, sT, st);
    return launch_tile<JET_SRC_BF16, true, false, true>(w, nullptr, N, K, q, s, qT, sT, st);
}

}  // namespace jet
