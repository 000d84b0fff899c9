// A 128x128 tile in the registers of a workgroup, quantized along its rows and along its columns: what the tile
// quantizer and the operators that quantize their result where it is formed share.
#pragma once

#include "jet_numerics.h"

namespace jet {

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

// LDS of a tile's maxima, column scales and transposed bytes
struct TileLds {
    float red[4 * 128];              // maxima of a wave's rows (BLOCK: one per wave)
    float2 scS[128];                 // S and 1/S of a column
    uint8_t T[128 * 128];
};

// Transposed row kl holds column k0 + kl of the tile along m: written out 16 B at a time.
__device__ __forceinline__ void store_transposed(TileLds& L, long m0, long k0, long M, uint8_t* __restrict__ q_colT) {
    const int t = threadIdx.x;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int kl = (t + 256 * i) >> 3, part = t & 7;
        *reinterpret_cast<uint4*>(q_colT + (k0 + kl) * M + m0 + 16 * part) =
            *reinterpret_cast<const uint4*>(&L.T[t_addr(kl, part)]);
    }
}

// Row and/or column quantization of the 128x128 tile at (m0, k0) of an [M, K] array; thread (rr = t >> 4, cc = t & 15) of 256 holds
// rows 8 rr .. and columns 8 cc .. .  Every thread of the workgroup calls it; a second call needs no barrier in between: what
// the first reads from the LDS last, T, the second writes behind two barriers.
template <ValueKind kKind, bool ROW, bool COL>
__device__ __forceinline__ void quantize_tile(const float (&v)[8][8], TileLds& L, long m0, long k0, long M, long K,
                                              uint8_t* __restrict__ q_row, float* __restrict__ s_row,
                                              uint8_t* __restrict__ q_colT, float* __restrict__ s_colT) {
    const int t = threadIdx.x, rr = t >> 4, cc = t & 15, w = t >> 6;
    const long GK = K / kGroup, GM = M / kGroup, gk = k0 / kGroup, gm = m0 / kGroup;
    if (COL) {
        float cm[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            cm[j] = 0.0f;
#pragma unroll
            for (int p = 0; p < 8; ++p) cm[j] = fmaxf(cm[j], fabsf(v[p][j]));
        }
        *reinterpret_cast<float2*>(&L.red[w * 128 + 8 * cc + 2 * (rr & 3)]) = wave_max_of_8(cm);
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
        if (cc < 8) s_row[(m0 + 8 * rr + cc) * GK + gk] = mine.S;
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
            const GroupScale gs = make_scale(fmaxf(fmaxf(L.red[t], L.red[128 + t]), fmaxf(L.red[256 + t], L.red[384 + t])));
            L.scS[t] = float2{gs.S, gs.r};
            s_colT[(k0 + t) * GM + gm] = gs.S;
            plain = gs.plain;
        }
        plain = __syncthreads_and(plain);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float2 sr = L.scS[8 * cc + j];
            const float c[8] = {v[0][j], v[1][j], v[2][j], v[3][j], v[4][j], v[5][j], v[6][j], v[7][j]};
            uint32_t o[2];
            encode<kKind>(c, GroupScale{sr.x, sr.y, plain}, o);
            *reinterpret_cast<uint2*>(&L.T[t_addr(8 * cc + j, rr >> 1) + 8 * (rr & 1)]) = uint2{o[0], o[1]};
        }
    }
    if (COL) store_transposed(L, m0, k0, M, q_colT);
}

}  // namespace jet
