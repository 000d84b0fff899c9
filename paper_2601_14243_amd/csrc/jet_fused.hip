// Fused producers: the operator in front of a GEMM writes its output directly as
// 1x128-quantized FP8 (Jet-RL Sec. 4.2: the activation quantization is fused with the
// previous operator; Sec. 4.3 names RMSNorm and the activation function).  The operator's
// bf16 result h is never stored: it is rounded to bf16 in registers and quantized with the
// row quantizer's arithmetic (jet_numerics.h), so the FP8 bytes and scales equal those of
// "operator in bf16, then jet_quant_act".  Both kernels are HBM-bound streams.
#include <algorithm>

#include "jet_internal.h"
#include "jet_numerics.h"
#include "jet_tile_quant.h"

namespace jet {

// ------------------------------------------------------------------------
// bf16 of a binary64 value with one rounding (finite input).  The conversion to binary32
// is monotonic, so the binary32 value lies on the same side of every bf16 tie point as the
// binary64 one -- unless it landed exactly on a tie, where the binary64 value decides.
// ------------------------------------------------------------------------
__device__ __forceinline__ uint32_t bf16_from_double(double v) {
    const float f = (float)v;
    const uint32_t u = __float_as_uint(f);
    if ((u & 0xffffu) == 0x8000u) {
        const double fd = (double)f;
        if (fd != v) return (u >> 16) + (fabs(v) > fabs(fd) ? 1u : 0u);
    }
    return bf16_rne(f);
}

// silu(g) = g / (1 + e^-g) of a bf16 value g with |g| <= 80, to be rounded to bf16.
// e^-g = 2^y with y = -g log2(e) split as -g c_hi (exact: 8 x 16 significant bits) plus a small remainder folded in
// as a factor 1 + ln2 * (-g c_lo); the hardware 2^y and reciprocal are good to 1 ulp each, and one residual
// correction of the quotient leaves it within 3 half ulps of the real value.  That is not a proof for the rounding to bf16, but
// the function has one 16-bit input: its bf16 rounding equals that of the binary64 evaluation for every finite g >= -87
// (the tests run all of them), so nothing has to be decided at run time.  The residual's sign keeps that of a zero input.
struct Silu {
    float a, e, r;    // silu(g), e^-g, 1 / (1 + e^-g)
};
__device__ __forceinline__ Silu silu_fast(float g) {
    const float c_hi = 0x1.7154p+0f, c_lo = 0x1.d94aep-18f, ln2 = 0x1.62e43p-1f;
    const float p2 = __builtin_amdgcn_exp2f(-g * c_hi);
    const float e = __builtin_fmaf(p2, (-g * c_lo) * ln2, p2);     // within 4 ulp
    const float d = 1.0f + e, r = __builtin_amdgcn_rcpf(d);
    const float q = g * r;
    return Silu{__builtin_fmaf(-__builtin_fmaf(d, q, -g), r, q), e, r};
}
constexpr float kSiluRange = 80.0f;
// the same rounded to bf16, for any finite g
__device__ __forceinline__ uint32_t silu_any(float g) {
    const double gd = (double)g;
    return bf16_from_double(gd / (1.0 + exp(-gd)));
}
// quantize the 16 values of a lane (a team of 8 lanes holds one 128-group) and store them
__device__ __forceinline__ void quantize_store(float (&v)[16], uint8_t* q16, float* s1, bool leader) {
    float am = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) am = fmaxf(am, fabsf(v[i]));
    am = team8_max(am);
    const GroupScale gs = make_scale(am);
    uint32_t o[4];
    encode<kBf16Values>(v, gs, o);
    *reinterpret_cast<uint4*>(q16) = uint4{o[0], o[1], o[2], o[3]};
    if (leader) *s1 = gs.S;
}

template <bool kNt = false>
__device__ __forceinline__ void unpack16(const uint16_t* p, float (&v)[16]) {
    const uint4* p4 = reinterpret_cast<const uint4*>(p);
    const uint4 u0 = kNt ? load16_nt(p4) : p4[0], u1 = kNt ? load16_nt(p4 + 1) : p4[1];
    const uint32_t w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[2 * i] = bf16_lo(w[i]);
        v[2 * i + 1] = bf16_hi(w[i]);
    }
}

// ------------------------------------------------------------------------
// SiLU(gate) * up -> 1x128 FP8.  a = bf16(silu(g)), h = bf16(a * u) (binary32 product).
// Same decomposition as the row quantizer: a team of 8 lanes owns a group, a lane 16
// consecutive elements (2 x 32 B in, 16 B out).  gate and up share the row stride ld.
// At memory speed for large calls ([16384, 14336]: 5.0 TB/s) once no value near a rounding tie went through binary64 (one
// gate in a thousand, -3.046875, did, and with it most waves): captured back to back, [1000, 14336] 16.6 -> 14.4 us,
// [8, 14336] 4.1 -> 2.9.
// ------------------------------------------------------------------------
template <bool kNt>
__global__ __launch_bounds__(256) void silu_mul_quant_kernel(const uint16_t* __restrict__ gate,
                                                             const uint16_t* __restrict__ up, long ld,
                                                             int groups_per_row, long n_groups,
                                                             uint8_t* __restrict__ q, float* __restrict__ s) {
    const long n_teams = (long)gridDim.x * 32;
    const int l8 = threadIdx.x & 7;
    for (long g = ((long)blockIdx.x * 256 + threadIdx.x) >> 3; g < n_groups; g += n_teams) {
        const long m = g / groups_per_row;
        const long src = m * ld + (g - m * groups_per_row) * kGroup + l8 * 16;
        float a[16], u[16], gmax = 0.0f;
        unpack16<kNt>(gate + src, a);
        unpack16<kNt>(up + src, u);
#pragma unroll
        for (int i = 0; i < 16; ++i) gmax = fmaxf(gmax, fabsf(a[i]));
        uint32_t act[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) act[i] = bf16_pack2(silu_fast(a[2 * i]).a, silu_fast(a[2 * i + 1]).a);
        if (!(gmax <= kSiluRange)) {    // one branch for the lane's 16 values, then only those out of range
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (fabsf(a[i]) <= kSiluRange) continue;
                const int sh = 16 * (i & 1);
                act[i >> 1] = (act[i >> 1] & (0xffffu << (16 - sh))) | (silu_any(a[i]) << sh);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t h2 = bf16_pack2(bf16_lo(act[i]) * u[2 * i], bf16_hi(act[i]) * u[2 * i + 1]);
            a[2 * i] = bf16_lo(h2);
            a[2 * i + 1] = bf16_hi(h2);
        }
        quantize_store(a, q + g * kGroup + l8 * 16, s + g, l8 == 0);
    }
}

// ------------------------------------------------------------------------
// RMSNorm -> 1x128 FP8.
//   1. sum of squares in binary64 (the square of a bf16 value is exact there); mean rounded once
//      to binary32; r = 1 / sqrt(mean + eps) in binary32;
//   2. n = bf16(x r), h = bf16(gamma n), quantized per 128-group.
// Rows up to 8192 columns add their squares in one order whatever kernel runs, so that a row's bytes do not
// depend on the batch it is in: a piece = 8 columns, ascending; lane i of 64 takes the pieces 2i and 2i+1 of
// every 1024 columns, ascending; then the 64 lanes by wave_sum.
// ------------------------------------------------------------------------
__device__ __forceinline__ double double_of(uint32_t lo, uint32_t hi) {
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return v + double_of(lo, hi);
}
// sum over the 64 lanes, the same value in every lane: neighbours, then quads, octets, 16-lane rows and halves
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        v = double_of(lo[0], hi[0]) + double_of(lo[1], hi[1]);
    }
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        v = double_of(lo[0], hi[0]) + double_of(lo[1], hi[1]);
    }
    return v;
}
__device__ __forceinline__ float rms_factor(double ss, int K, float eps) {
    const float ms = (float)(ss / (double)K);
    return 1.0f / sqrtf(ms + eps);
}

__device__ __forceinline__ void unpack8(uint4 u, float (&v)[8]) {
    v[0] = bf16_lo(u.x); v[1] = bf16_hi(u.x);
    v[2] = bf16_lo(u.y); v[3] = bf16_hi(u.y);
    v[4] = bf16_lo(u.z); v[5] = bf16_hi(u.z);
    v[6] = bf16_lo(u.w); v[7] = bf16_hi(u.w);
}
__device__ __forceinline__ double piece_of(const float* v) {
    double p = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) p = fma((double)v[i], (double)v[i], p);
    return p;
}

// A workgroup of K / 8 threads (whole waves) per row, one piece per thread (K <= 8192): for few rows, where a
// call is bound by its chain of latencies (launch, first loads, instruction fetch, reduction, division), not by bytes.
__global__ __launch_bounds__(1024) void rmsnorm_quant_row_kernel(const uint16_t* __restrict__ x,
                                                                 const uint16_t* __restrict__ gamma, float eps,
                                                                 int K, uint8_t* __restrict__ q,
                                                                 float* __restrict__ s) {
    __shared__ double2 pieces[512];
    const int t = threadIdx.x, l = t & 63;
    const long m = blockIdx.x;
    const int n_pieces = K >> 3;
    const bool mine = t < n_pieces;                      // whole 16-lane rows: K is a multiple of 128
    float v[8], gm[8];
    uint4 gu = {0, 0, 0, 0};
    if (mine) {
        const uint4 xu = *reinterpret_cast<const uint4*>(x + m * K + t * 8);
        gu = *reinterpret_cast<const uint4*>(gamma + t * 8);
        unpack8(xu, v);
        reinterpret_cast<double*>(pieces)[t] = piece_of(v);
    }
    __syncthreads();
    double ss = 0.0;
    for (int i = l; 2 * i < n_pieces; i += 64) {         // the 64 pairs of pieces of each 1024 columns
        const double2 p = pieces[i];
        ss += p.x;
        ss += p.y;
    }
    const float r = rms_factor(wave_sum(ss), K, eps);
    if (!mine) return;
    unpack8(gu, gm);
    float am = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const uint32_t n2 = bf16_pack2(v[i] * r, v[i + 1] * r);
        const uint32_t h2 = bf16_pack2(gm[i] * bf16_lo(n2), gm[i + 1] * bf16_hi(n2));
        v[i] = bf16_lo(h2);
        v[i + 1] = bf16_hi(h2);
        am = fmaxf(am, fmaxf(fabsf(v[i]), fabsf(v[i + 1])));
    }
    const GroupScale gs = make_scale(team16_max(am));
    uint32_t o[2];
    encode<kBf16Values>(v, gs, o);
    *reinterpret_cast<uint2*>(q + m * K + t * 8) = uint2{o[0], o[1]};
    if ((t & 15) == 0) s[m * (K >> 7) + (t >> 4)] = gs.S;
}

// A team of kTeam threads per row, which stays in registers (a thread holds 16-element chunks, one per
// 16 kTeam columns): kTeam = 64, a wave per row and four rows per workgroup without a barrier, for rows up
// to 8192 columns; kTeam = 256 (the workgroup, one barrier) beyond.
template <int kTeam, int MAXCH>
__global__ __launch_bounds__(256) void rmsnorm_quant_kernel(const uint16_t* __restrict__ x,
                                                            const uint16_t* __restrict__ gamma, float eps,
                                                            long M, int K, uint8_t* __restrict__ q,
                                                            float* __restrict__ s) {
    __shared__ double part[4];
    const int t = threadIdx.x, l8 = t & 7;
    const int lane = (kTeam == 64) ? (t & 63) : t;
    const long m = (kTeam == 64) ? (long)blockIdx.x * 4 + (t >> 6) : (long)blockIdx.x;
    if (m >= M) return;                                  // whole waves; only with a wave per row
    const uint16_t* row = x + m * K;
    float v[MAXCH][16];
    double ss = 0.0;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int k0 = (c * kTeam + lane) * 16;
        if (k0 < K) unpack16(row + k0, v[c]);
    }
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int k0 = (c * kTeam + lane) * 16;
        if (k0 < K) {
            ss += piece_of(v[c]);
            ss += piece_of(v[c] + 8);
        }
    }
    ss = wave_sum(ss);
    if (kTeam == 256) {
        if ((t & 63) == 0) part[t >> 6] = ss;
        __syncthreads();
        ss = (part[0] + part[1]) + (part[2] + part[3]);
    }
    const float r = rms_factor(ss, K, eps);
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int k0 = (c * kTeam + lane) * 16;
        if (k0 < K) {   // whole groups: 8 lanes hold one, and K is a multiple of 128
            float gm[16];
            unpack16(gamma + k0, gm);
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                const uint32_t n2 = bf16_pack2(v[c][i] * r, v[c][i + 1] * r);
                const uint32_t h2 = bf16_pack2(gm[i] * bf16_lo(n2), gm[i + 1] * bf16_hi(n2));
                v[c][i] = bf16_lo(h2);
                v[c][i + 1] = bf16_hi(h2);
            }
            quantize_store(v[c], q + m * K + k0, s + (m * K + k0) / kGroup, l8 == 0);
        }
    }
}

// ------------------------------------------------------------------------
// Backward of h = bf16(bf16(silu(g)) * u), the element-wise operator between the down projection
// and the gate/up projections of an MLP block (Sec. 4.1: gradients between operators stay bf16):
//   dup = bf16(dh * a),  da = bf16(dh * u),  dgate = bf16(da * silu'(g)),
//   a = bf16(silu(g)) as in the forward,  silu'(g) = s (1 + g (1 - s)),  s = 1 / (1 + e^-g).
// The two products of bf16 values are exact in binary32, so their bf16 rounding is the single
// rounding of the real value.  dgate is the real value da * silu'(g) rounded once: the binary32
// evaluation below carries an error bound (in ulps, growing towards the zero of silu' at
// g = -1.2785 where 1 + g (1 - s) cancels), and whenever the result is closer than that bound to
// a bf16 tie, or outside the range the bound holds in, binary64 decides.
// ------------------------------------------------------------------------
// With 2^y and the reciprocal good to 1 ulp: e within 4 ulp, s within 5, 1 - s within 9, w within 10 ulp(g om) and half an ulp of
// its own, so prod within 7 + 10 |g om| / |w| ulps.  The window is twice that: any error of one ulp either way in the two
// instructions, on any gate value, uses less than half of it (a CPU model of this function in the tests).  No intermediate value is
// subnormal for |g| <= 80 (r w is 2^-109 at least), so the bound holds for every normal product.  A zero da (the rows of masked
// tokens) gives a zero with the sign of silu', which w carries: binary64 for whole rows of them would make a call slower the more
// tokens are masked.  us at [4096, 14336] with none, a quarter, half, all of the rows zero: jet_silu_mul_bwd 109 / 155 / 178 / 246 with
// zeros in binary64, 106 / 108 / 110 / 106 now; jet_silu_mul_bwd_quant 196 / 221 / 244 / 292, 186 / 189 / 188 / 178 now.
__device__ __forceinline__ float silu_grad_mul(float g, float da, const Silu& s, bool& sure) {
    const float om = s.e * s.r;                                    // 1 - s without cancellation
    const float gom = g * om;
    const float w = 1.0f + gom;
    const float prod = da * (s.r * w);
    const float window = 16.0f + 24.0f * fabsf(gom) * __builtin_amdgcn_rcpf(fabsf(w));
    const float dist = fabsf((float)(int)(__float_as_uint(prod) & 0xffffu) - 32768.0f);
    sure = dist > window && fabsf(g) <= kSiluRange && (fabsf(prod) >= 0x1p-125f || da == 0.0f);
    return prod;
}
// the same rounded to bf16, for any finite g; od = 1 + e^-g
__device__ __forceinline__ uint32_t silu_grad_mul_any(double gd, double od, float da) {
    const double sd = 1.0 / od;
    return bf16_from_double((double)da * (sd * (1.0 + gd * (1.0 - sd))));
}

// eight neighbouring elements: dgate and dup as bf16
__device__ __forceinline__ void silu_mul_bwd8(const uint4 g4, const uint4 u4, const uint4 d4, uint32_t (&og)[4], uint32_t (&ou)[4]) {
    const uint32_t gw[4] = {g4.x, g4.y, g4.z, g4.w}, uw[4] = {u4.x, u4.y, u4.z, u4.w}, dw[4] = {d4.x, d4.y, d4.z, d4.w};
    uint32_t unsure = 0;            // bit per value: one branch for the thread's 8, then only what needs it
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float g0 = bf16_lo(gw[i]), g1 = bf16_hi(gw[i]);
        const float u0 = bf16_lo(uw[i]), u1 = bf16_hi(uw[i]);
        const float d0 = bf16_lo(dw[i]), d1 = bf16_hi(dw[i]);
        const Silu s0 = silu_fast(g0), s1 = silu_fast(g1);
        const uint32_t a2 = bf16_pack2(s0.a, s1.a);
        ou[i] = bf16_pack2(d0 * bf16_lo(a2), d1 * bf16_hi(a2));
        const uint32_t da2 = bf16_pack2(d0 * u0, d1 * u1);
        bool sure0, sure1;
        const float p0 = silu_grad_mul(g0, bf16_lo(da2), s0, sure0), p1 = silu_grad_mul(g1, bf16_hi(da2), s1, sure1);
        og[i] = bf16_pack2(p0, p1);
        unsure |= (sure0 ? 0u : 1u << (2 * i)) | (sure1 ? 0u : 2u << (2 * i));
    }
    // one copy of the binary64 code for the eight: a lane rarely has two such values
    while (unsure) {
        const int i = __builtin_ctz(unsure), w = i >> 1, sh = 16 * (i & 1);
        unsure &= unsure - 1;
        auto pick = [&](const uint32_t (&x)[4]) {       // by value: a choice between addresses would put x into memory
            const uint32_t lo = (w & 1) ? +x[1] : +x[0], hi = (w & 1) ? +x[3] : +x[2];
            return w < 2 ? +lo : +hi;
        };
        const uint32_t keep = 0xffffu << (16 - sh);
        const float g = __uint_as_float((pick(gw) >> sh) << 16), d = __uint_as_float((pick(dw) >> sh) << 16);
        const float u = __uint_as_float((pick(uw) >> sh) << 16);
        const double gd = (double)g, od = 1.0 + exp(-gd);
        const float da = __uint_as_float(bf16_rne(d * u) << 16);
        const uint32_t dg = (pick(og) & keep) | (silu_grad_mul_any(gd, od, da) << sh);
        uint32_t du = pick(ou);
        if (!(fabsf(g) <= kSiluRange))
            du = (du & keep) | (bf16_rne(d * __uint_as_float(bf16_from_double(gd / od) << 16)) << sh);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            og[j] = w == j ? dg : og[j];
            ou[j] = w == j ? du : ou[j];
        }
    }
}

__global__ __launch_bounds__(256) void silu_mul_bwd_kernel(const uint16_t* __restrict__ gate,
                                                           const uint16_t* __restrict__ up, long ld,
                                                           const uint16_t* __restrict__ dh, int chunks_per_row,
                                                           long n_chunks, uint16_t* __restrict__ dgate,
                                                           uint16_t* __restrict__ dup, long ld_out) {
    const long stride = (long)gridDim.x * 256;
    for (long c = (long)blockIdx.x * 256 + threadIdx.x; c < n_chunks; c += stride) {
        const long m = c / chunks_per_row;
        const long k = (c - m * chunks_per_row) * 8;
        uint32_t og[4], ou[4];
        silu_mul_bwd8(*reinterpret_cast<const uint4*>(gate + m * ld + k), *reinterpret_cast<const uint4*>(up + m * ld + k),
                      *reinterpret_cast<const uint4*>(dh + m * (long)chunks_per_row * 8 + k), og, ou);
        *reinterpret_cast<uint4*>(dgate + m * ld_out + k) = uint4{og[0], og[1], og[2], og[3]};
        *reinterpret_cast<uint4*>(dup + m * ld_out + k) = uint4{ou[0], ou[1], ou[2], ou[3]};
    }
}

// The same and, from registers, the row and column quantization of [dgate | dup] for the gate/up DGrad and WGrad: the bf16
// gradient is written once and not read back.  A workgroup forms a 128x128 tile of dgate and the one of dup beside it and
// quantizes them in turn; the arithmetic is that of silu_mul_bwd_kernel and of the tile quantizer, so the bytes are
// theirs.  Bound by HBM: 14.1 bytes per element of dh instead of 18.1 in two launches.  All 24 loads of a thread go out
// first; nobody reads gate, up, dh and dgu again soon, so they pass the memory-side cache.  Captured, us: [16384, 14336] two launches 880, this
// 726; small calls lose by it ([512, 3072] 13.4 -> 18.8: the caller has the line).
__global__ __launch_bounds__(256) void silu_mul_bwd_quant_kernel(const uint16_t* __restrict__ gate,
                                                                 const uint16_t* __restrict__ up, long ld,
                                                                 const uint16_t* __restrict__ dh, long M, long K,
                                                                 uint16_t* __restrict__ dgu, uint8_t* __restrict__ q_row,
                                                                 float* __restrict__ s_row, uint8_t* __restrict__ q_colT,
                                                                 float* __restrict__ s_colT) {
    __shared__ __attribute__((aligned(16))) TileLds L;
    const int t = threadIdx.x, rr = t >> 4, cc = t & 15;
    const long m0 = (long)blockIdx.y * 128, k0 = (long)blockIdx.x * 128, k = k0 + 8 * cc;
    uint4 g4[8], u4[8], d4[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const long m = m0 + 8 * rr + p;
        g4[p] = load16_nt(gate + m * ld + k);
        u4[p] = load16_nt(up + m * ld + k);
        d4[p] = load16_nt(dh + m * K + k);
    }
    uint32_t og[8][4], ou[8][4];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        silu_mul_bwd8(g4[p], u4[p], d4[p], og[p], ou[p]);
        uint16_t* row = dgu + (m0 + 8 * rr + p) * 2 * K + k;
        store16_nt(row, uint4{og[p][0], og[p][1], og[p][2], og[p][3]});
        store16_nt(row + K, uint4{ou[p][0], ou[p][1], ou[p][2], ou[p][3]});
    }
    auto quantize = [&](const uint32_t (&h)[8][4], long col) {
        float v[8][8];
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[p][2 * i] = bf16_lo(h[p][i]);
                v[p][2 * i + 1] = bf16_hi(h[p][i]);
            }
        quantize_tile<kBf16Values, true, true>(v, L, m0, col, M, 2 * K, q_row, s_row, q_colT, s_colT);
    };
    quantize(og, k0);
    quantize(ou, K + k0);
}

// ----------------------------------------------------------------- launch --

hipError_t launch_silu_mul_quant(const void* gate, const void* up, long ld, long M, long K, uint8_t* q,
                                 float* s, hipStream_t st) {
    const long n_groups = M * (K / kGroup);
    const long blocks = std::min<long>((n_groups + 31) / 32, 256L * 64);
    // An input larger than the 256 MB memory-side cache is not in it any more when it is read, and reading it past that cache
    // leaves the codes there for the down projection: [16384, 14336] 230 -> 221 us, with that GEMM 1067 -> 1041, [8192, 14336]
    // 520 -> 510.  Smaller inputs, which the gate/up GEMM has just written, lose by it (1000 rows with the GEMM 92.7 -> 94.5).
    const auto kernel = 4 * M * K > (256L << 20) ? silu_mul_quant_kernel<true> : silu_mul_quant_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint16_t*>(gate), static_cast<const uint16_t*>(up), ld,
                       (int)(K / kGroup), n_groups, q, s);
    return hipGetLastError();
}

hipError_t launch_silu_mul_bwd(const void* gate, const void* up, long ld, const void* dh, long M, long K,
                               void* dgate, void* dup, long ld_out, hipStream_t st) {
    const long n_chunks = M * (K / 8);
    const long blocks = std::min<long>((n_chunks + 255) / 256, 256L * 32);
    hipLaunchKernelGGL(silu_mul_bwd_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint16_t*>(gate), static_cast<const uint16_t*>(up), ld,
                       static_cast<const uint16_t*>(dh), (int)(K / 8), n_chunks,
                       static_cast<uint16_t*>(dgate), static_cast<uint16_t*>(dup), ld_out);
    return hipGetLastError();
}

hipError_t launch_silu_mul_bwd_quant(const void* gate, const void* up, long ld, const void* dh, long M, long K, void* dgu,
                                     uint8_t* q_row, float* s_row, uint8_t* q_colT, float* s_colT, hipStream_t st) {
    hipLaunchKernelGGL(silu_mul_bwd_quant_kernel, dim3((unsigned)(K / 128), (unsigned)(M / 128)), dim3(256), 0, st,
                       static_cast<const uint16_t*>(gate), static_cast<const uint16_t*>(up), ld,
                       static_cast<const uint16_t*>(dh), M, K, static_cast<uint16_t*>(dgu), q_row, s_row, q_colT, s_colT);
    return hipGetLastError();
}

hipError_t launch_rmsnorm_quant(const void* x, const void* gamma, float eps, long M, long K, uint8_t* q,
                                float* s, hipStream_t st) {
    const uint16_t* xp = static_cast<const uint16_t*>(x);
    const uint16_t* gp = static_cast<const uint16_t*>(gamma);
#define JET_RMS(TEAM, N, GRID) \
    hipLaunchKernelGGL((rmsnorm_quant_kernel<TEAM, N>), dim3((unsigned)(GRID)), dim3(256), 0, st, xp, gp, eps, M, (int)K, q, s)
    // Few rows: a wave per row would leave its CU with one wave that runs 64 elements and 8 KB of cold
    // instructions one after the other.  4096 columns, captured back to back: 6.2 -> 2.8 us at 8 rows, 6.3 -> 3.2 at
    // 256, 6.8 -> 5.8 at 1000; at 2048 rows the barrier costs more than it gives (9.7 against 8.7).
    if (K <= 8192 && M <= 1024) {
        const unsigned threads = (unsigned)((K / 8 + 63) / 64 * 64);
        hipLaunchKernelGGL(rmsnorm_quant_row_kernel, dim3((unsigned)M), dim3(threads), 0, st, xp, gp, eps, (int)K, q, s);
        return hipGetLastError();
    }
    if (K <= 8192) {
        const int chunks = (int)((K + 1023) / 1024);
        const long grid = (M + 3) / 4;
        if (chunks <= 1) JET_RMS(64, 1, grid);
        else if (chunks <= 2) JET_RMS(64, 2, grid);
        else if (chunks <= 4) JET_RMS(64, 4, grid);
        else JET_RMS(64, 8, grid);
    } else {
        const int chunks = (int)((K + 4095) / 4096);
        if (chunks <= 4) JET_RMS(256, 4, M);
        else JET_RMS(256, 8, M);
    }
#undef JET_RMS
    return hipGetLastError();
}

}  // namespace jet
