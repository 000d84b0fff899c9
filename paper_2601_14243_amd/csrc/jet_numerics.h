// Device-side numerics contract of libjet (gfx950 only).
//
// Everything that decides an output bit lives here, so that every kernel --
// decode-shaped or training-shaped -- takes the same decisions:
//   * the quantizer step  S = amax/448, t = x/S (IEEE binary32), E4M3 RNE with
//     saturation (Jet-RL Sec. 2.1);
//   * the GEMM element chain: one FP8 MFMA over the 128 products of a group,
//     s = sa*sb, acc = fma(p, s, acc), groups ascending, bf16 RNE at the end
//     (Sec. 2.2 on the 1x128 / 128x128 operands of Sec. 4.2);
//   * the assignment of the 128 bytes of a group to MFMA lanes and registers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jet {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kGroup = 128;          // quantization group length (Sec. 4.2)
constexpr float kDeltaMax = 448.0f;  // largest finite E4M3 value (Sec. 2.1)

// ------------------------------------------------------------------ bf16 --

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// binary32 -> bf16, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// two floats -> two bf16 (round to nearest even) in one dword, low half first: one
// hardware convert for the pair
__device__ __forceinline__ uint32_t bf16_pack2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Loads of lines that are not needed again: they leave the 256 MB memory-side cache to what is.
__device__ __forceinline__ uint4 load16_nt(const void* p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(static_cast<const u32x4*>(p)));
}
__device__ __forceinline__ void store16_nt(void* p, uint4 v) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), static_cast<u32x4*>(p));
}
__device__ __forceinline__ uint2 load8_nt(const void* p) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint2, __builtin_nontemporal_load(static_cast<const u32x2*>(p)));
}

// ------------------------------------------------------------- quantizer --

// Scale of a group and the data needed to divide by it.
struct GroupScale {
    float S;     // amax / 448, or 1 for an all-zero group
    float r;     // correctly rounded 1/S
    bool plain;  // S far from the binary32 range limits
};

__device__ __forceinline__ GroupScale make_scale(float amax) {
    GroupScale g;
    g.S = (amax == 0.0f) ? 1.0f : amax / kDeltaMax;  // IEEE division
    g.plain = (g.S >= 0x1p-80f) && (g.S <= 0x1p80f);
    g.r = 1.0f / g.S;                                // IEEE division
    return g;
}

// Where the values of a group come from, which decides how much of the division they need.
enum ValueKind { kBf16Values, kFloatValues };

// Four values of a group of plain scale -> four E4M3 codes (little-endian): the E4M3 rounding of
// t = RN(x / S).  With r = RN(1/S), q0 = RN(x r) and an fma residual correction, q1 is RN of x/S moved by less than
// 2^-22 ulp; a second correction gives RN(x/S) itself (Markstein's division theorem), as long as nothing leaves the
// normal range, which a plain scale guarantees for every t that can round to a non-zero code.  q1 and t can only
// round to different codes if x/S lies within 2^-22 ulp of half an ulp beside an E4M3 rounding boundary: no pair of a
// bf16 x and the bf16 amax of its group does (the tests run every such pair through the row and the tile quantizer),
// so one correction does for bf16 values; binary32 values take both.
// The residual has the sign of q S - x, so that a zero input keeps its sign: -(+0) r + (-0) = -0.
// |t| <= 448 (1 + 2^-22), which rounds to 448: the convert (round to nearest even, also into the subnormal
// range, sign of zero kept, no saturation: NaN beyond 464) needs no clamp here.
template <ValueKind kKind>
__device__ __forceinline__ uint32_t codes4(float a, float b, float c, float d, float S, float r) {
    float x[4] = {a, b, c, d}, q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        q[i] = x[i] * r;
        q[i] = __builtin_fmaf(-__builtin_fmaf(q[i], S, -x[i]), r, q[i]);
        if (kKind == kFloatValues) q[i] = __builtin_fmaf(-__builtin_fmaf(q[i], S, -x[i]), r, q[i]);
    }
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], w, true);
    return (uint32_t)w;
}

// The same for any scale: IEEE division, clamp to +-448 (a subnormal S may be off by more than 3 %; every value in
// (448, 464) rounds to 448 anyway), convert.
__device__ __forceinline__ uint32_t codes4_any(float a, float b, float c, float d, float S) {
    float x[4] = {a, b, c, d};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        x[i] = __builtin_amdgcn_fmed3f(__builtin_copysignf(x[i] / S, x[i]), -kDeltaMax, kDeltaMax);
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], w, true);
    return (uint32_t)w;
}

// N values of one group -> N / 4 words of codes.  One branch per group and not per element, so that the
// elements' chains overlap.
template <ValueKind kKind, int N>
__device__ __forceinline__ void encode(const float (&v)[N], const GroupScale& g, uint32_t (&o)[N / 4]) {
    if (g.plain) {
#pragma unroll
        for (int i = 0; i < N; i += 4) o[i / 4] = codes4<kKind>(v[i], v[i + 1], v[i + 2], v[i + 3], g.S, g.r);
    } else {
#pragma unroll
        for (int i = 0; i < N; i += 4) o[i / 4] = codes4_any(v[i], v[i + 1], v[i + 2], v[i + 3], g.S);
    }
}

// Four E4M3 codes of one dword -> binary32 (exact).
__device__ __forceinline__ void e4m3_unpack4(uint32_t w, float& a, float& b, float& c, float& d) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
    v2f hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
    a = lo[0]; b = lo[1]; c = hi[0]; d = hi[1];
}

// max of non-negative floats (never NaN: they start from 0 through fmaxf), compared as integers so that the
// lane permutation folds into the instruction
__device__ __forceinline__ float max_nonneg(float a, float b) {
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float(x > y ? x : y);
}
// max over a team of 8 / 16 consecutive lanes (all lanes of the team get it).
template <int CTRL>
__device__ __forceinline__ float dpp_max(float v) {
    return max_nonneg(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ float team8_max(float v) {
    v = dpp_max<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_max<0x4E>(v);   // quad_perm [2,3,0,1]
    v = dpp_max<0x141>(v);  // row_half_mirror
    return v;
}
__device__ __forceinline__ float team16_max(float v) {
    v = team8_max(v);
    v = dpp_max<0x140>(v);  // row_mirror
    return v;
}

// ------------------------------------------------------------------ GEMM --

// MFMA operand fragment of one 16-row x 128-byte group tile.  Lane l serves
// row (l & 15) and 16-byte chunk column c4 = l >> 4: registers 0-3 hold bytes
// [16 c4, 16 c4 + 16) and registers 4-7 hold bytes [64 + 16 c4, 64 + 16 c4 + 16)
// of that row's 128-byte group.  Every kernel loads both operands this way, so
// a given pair of rows always meets the matrix core in the same arrangement.
__device__ __forceinline__ v8i make_frag(uint4 lo, uint4 hi) {
    v8i f = {(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    return f;
}

// Partial sums of one group for a 16x16 output tile of OUT[i,j] = sum_r A[i,r] B[j,r]:
// p[t] belongs to (B row 4*(lane>>4)+t, A row lane&15).  The operand that indexes
// output columns (the weight in FProp and DGrad, X^T in WGrad) always goes first and
// the operand that indexes output rows second, in every kernel.
__device__ __forceinline__ v4f group_product(v8i col_frag, v8i row_frag) {
    v4f z = {0.0f, 0.0f, 0.0f, 0.0f};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(col_frag, row_frag, z, 0, 0, 0, 0, 0, 0);
}

// One step of the scaled accumulation chain.
__device__ __forceinline__ float chain(float p, float s, float acc) { return __builtin_fmaf(p, s, acc); }

// s_waitcnt vmcnt(n) with the other counters left alone (gfx9 encoding).
#define JET_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xf) | (((n) >> 4) << 14) | (0x7 << 4) | (0xf << 8))

}  // namespace jet
