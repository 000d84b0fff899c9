// Fused amax / scale / cast quantizers (Jet-RL Sec. 2.1 formula at the
// granularities of Sec. 4.2).  All of them are HBM-bound streaming kernels:
// every input byte is read once with 16-byte loads, every output byte written
// once, reductions stay in registers (DPP) or LDS.
#include "jet_internal.h"
#include "jet_numerics.h"

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

// broadcast of lane N of every 16-lane row
template <int N>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 | N, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// a[p] of the 16 lanes of a row -> their max; lane i of the row gets that of p = i & 7.  Halving: lanes that
// differ in bit 0 (then bit 1) exchange half of their values, the rest by rotation.
__device__ __forceinline__ float row_max_of_8(const float (&a)[8], int lane) {
    const bool odd = lane & 1, hi = lane & 2;
    float b[4], c[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        b[i] = max_nonneg(odd ? a[2 * i + 1] : a[2 * i], dpp_move<0xB1>(odd ? a[2 * i] : a[2 * i + 1]));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        c[i] = max_nonneg(hi ? b[2 * i + 1] : b[2 * i], dpp_move<0x4E>(hi ? b[2 * i] : b[2 * i + 1]));
        c[i] = dpp_max<0x124>(c[i]);   // row_ror:4
        c[i] = dpp_max<0x128>(c[i]);   // row_ror:8
    }
    return (lane & 4) ? c[1] : c[0];
}
// a[j] of the four 16-lane rows -> their max; row q gets that of j = 2q and 2q + 1
__device__ __forceinline__ float2 wave_max_of_8(const float (&a)[8]) {
    float b[4], c[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(a[i + 4]), false, false);
        b[i] = max_nonneg(__uint_as_float(w[0]), __uint_as_float(w[1]));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[i]), __float_as_uint(b[i + 2]), false, false);
        c[i] = max_nonneg(__uint_as_float(w[0]), __uint_as_float(w[1]));
    }
    return float2{c[0], c[1]};
}
// byte e of o[j] = byte j of argument e
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&o)[4]) {
    const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602);
    const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602);
    o[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100);
    o[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302);
    o[2] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100);
    o[3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302);
}
// LDS address of the 16-byte chunk `chunk` of transposed row `row` (128 bytes per row): a wave writes one
// row in 8, 8 bytes each, and reads whole rows, both without a bank conflict
__device__ __forceinline__ int t_addr(int row, int chunk) {
    return (row ^ ((row >> 3) & 1)) * 128 + 16 * (chunk ^ ((row >> 3) & 7));
}

template <int SRC, bool ROW, bool COL, bool BLOCK>
__global__ __launch_bounds__(256) void quant_tile_kernel(const void* __restrict__ x,
                                                         const float* __restrict__ xs, long M, long K,
                                                         uint8_t* __restrict__ q_row,
                                                         float* __restrict__ s_row,
                                                         uint8_t* __restrict__ q_colT,
                                                         float* __restrict__ s_colT) {
    constexpr ValueKind kKind = SRC == JET_SRC_BF16 ? kBf16Values : kFloatValues;
    __shared__ __attribute__((aligned(16))) float red[4 * 128];      // maxima of a wave's rows (BLOCK: one per wave)
    __shared__ __attribute__((aligned(16))) float2 scS[128];         // S and 1/S of a column
    __shared__ __attribute__((aligned(16))) uint8_t T[128 * 128];

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
        if ((t & 63) == 0) red[w] = am;
        __syncthreads();
        am = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
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
                    *reinterpret_cast<uint2*>(&T[t_addr(8 * cc + 4 * h + j, rr >> 1) + 8 * (rr & 1)]) = uint2{up[j], dn[j]};
            }
        }
    } else {
        if (COL) {
            float cm[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                cm[j] = 0.0f;
#pragma unroll
                for (int p = 0; p < 8; ++p) cm[j] = fmaxf(cm[j], fabsf(v[p][j]));
            }
            *reinterpret_cast<float2*>(&red[w * 128 + 8 * cc + 2 * (rr & 3)]) = wave_max_of_8(cm);
        }
        if (ROW) {
            float am[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                am[p] = 0.0f;
#pragma unroll
                for (int j = 0; j < 8; ++j) am[p] = fmaxf(am[p], fabsf(v[p][j]));
            }
            // lane cc forms the scale of row cc & 7 of its thread row
            const GroupScale mine = make_scale(row_max_of_8(am, cc));
            if (cc < 8) s_row[(m0 + 8 * rr + cc) * GK + blockIdx.x] = mine.S;
            const float S[8] = {row_bcast<0>(mine.S), row_bcast<1>(mine.S), row_bcast<2>(mine.S), row_bcast<3>(mine.S),
                                row_bcast<4>(mine.S), row_bcast<5>(mine.S), row_bcast<6>(mine.S), row_bcast<7>(mine.S)};
            const float r[8] = {row_bcast<0>(mine.r), row_bcast<1>(mine.r), row_bcast<2>(mine.r), row_bcast<3>(mine.r),
                                row_bcast<4>(mine.r), row_bcast<5>(mine.r), row_bcast<6>(mine.r), row_bcast<7>(mine.r)};
            const bool plain = __all(mine.plain);            // of the wave's 32 rows
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                uint32_t o[2];
                encode<kKind>(v[p], GroupScale{S[p], r[p], plain}, o);
                *reinterpret_cast<uint2*>(q_row + (m0 + 8 * rr + p) * K + k0 + 8 * cc) = uint2{o[0], o[1]};
            }
        }
        if (COL) {
            __syncthreads();
            bool plain = true;
            if (t < 128) {
                const GroupScale gs = make_scale(fmaxf(fmaxf(red[t], red[128 + t]), fmaxf(red[256 + t], red[384 + t])));
                scS[t] = float2{gs.S, gs.r};
                s_colT[(k0 + t) * GM + blockIdx.y] = gs.S;
                plain = gs.plain;
            }
            plain = __syncthreads_and(plain);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float2 sr = scS[8 * cc + j];
                const float c[8] = {v[0][j], v[1][j], v[2][j], v[3][j], v[4][j], v[5][j], v[6][j], v[7][j]};
                uint32_t o[2];
                encode<kKind>(c, GroupScale{sr.x, sr.y, plain}, o);
                *reinterpret_cast<uint2*>(&T[t_addr(8 * cc + j, rr >> 1) + 8 * (rr & 1)]) = uint2{o[0], o[1]};
            }
        }
    }

    if (COL) {
        __syncthreads();
        // transposed row kl holds column k0+kl of the tile along m: write it out 16 B at a time
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kl = (t + 256 * i) >> 3, part = t & 7;
            *reinterpret_cast<uint4*>(q_colT + (k0 + kl) * M + m0 + 16 * part) =
                *reinterpret_cast<const uint4*>(&T[t_addr(kl, part)]);
        }
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
