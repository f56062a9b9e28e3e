// sre2_tile.h - the register/LDS tile engine of the fused and two-pass kernels:
// plan selection, the split forms' H_16 factors on the matrix cores, and the
// rounds of a transform.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sre2_plan.h"
#include "sre2_geometry.h"
#include "sre2_internal.h"
#include "sre2_device.h"

namespace sre2 {

#ifndef SRE2_SPLIT_P1_TAIL
#define SRE2_SPLIT_P1_TAIL 1  // split-form pass 1 ends in a store-layout round
#endif
// Minimum waves per SIMD asked of the compiler (register budget 512 / waves).
// Split-form pass 1 on 2^12 rows keeps its MFMA results in VGPRs at 3 (with
// fewer, the compiler moves them through AGPRs, which costs it about half its
// speed); LDS limits every TB = 12 kernel to 2.5 waves per SIMD anyway, and
// longer rows to 2.  Split-form pass 2 cannot reach 3 without spilling and is
// left alone.
#ifndef SRE2_P1_WAVES
#define SRE2_P1_WAVES 1
#endif
#ifndef SRE2_P1S_WAVES
#define SRE2_P1S_WAVES 3  // split form
#endif
#ifndef SRE2_P2_WAVES
#define SRE2_P2_WAVES 1
#endif
#ifndef SRE2_P2S_WAVES
#define SRE2_P2S_WAVES 1
#endif
#ifndef SRE2_FUSED_WAVES
#define SRE2_FUSED_WAVES 1
#endif
#ifndef SRE2_FUSEDS_WAVES
#define SRE2_FUSEDS_WAVES 2
#endif
// Half-LDS tiles: two workgroups share a CU.  They ask for the waves per SIMD
// that takes (half_waves: four for 512-thread FP32 tiles, i.e. at most 128
// registers, two for 256-thread FP64 tiles).
#ifndef SRE2_HALF_WGS
#define SRE2_HALF_WGS 2  // workgroups per CU that half-LDS two-pass tiles aim for
#endif
// Waves per SIMD that SRE2_HALF_WGS workgroups of 2^(TB - RB) threads need
// (four SIMDs per CU, 64 lanes per wave): the register budget per wave.
__host__ __device__ constexpr int half_waves(int tb, int rb) {
    const int w = SRE2_HALF_WGS * (1 << (tb - rb)) / 256;
    return w < 1 ? 1 : w;
}
// Plan selector (PK encodes the kind so that plans stay constexpr):
//   PK = 1000 + N : whole transform over tile bits [0, N)        (fused)
//   PK = 2000     : row transform over all TB tile bits          (pass 1)
//   PK = 3000 + H : column transform over the top H tile bits    (pass 2)
//   PK + 10000 s  : the same transform in split form s (1: FP16, 2: BF16
//                   halves; one plan for both), with H_16 factors on the
//                   matrix cores (pass 1 ends with a round whose lanes run
//                   over the lowest bits, for the stores)
//   two-pass tiles above 64 KiB (half_lds) take half-LDS plans
template <typename Real, int TB, int RB, int PK>
__host__ __device__ constexpr Plan plan_of() {
    constexpr int SB = Prec<Real>::SB;
    constexpr bool H = half_lds<Real>(TB);
    if (PK >= 10000) {
        constexpr int K = PK % 10000;
        if (K >= 3000)
            return H ? make_split_plan_half(TB, RB, SB, TB - (K - 3000), 0)
                     : make_split_plan(TB, RB, SB, TB - (K - 3000), TB, 0);
        if (K >= 2000)
            return H ? make_split_plan_half(TB, RB, SB, 0, SRE2_SPLIT_P1_TAIL)
                     : make_split_plan(TB, RB, SB, 0, TB, SRE2_SPLIT_P1_TAIL);
        return make_split_plan(TB, RB, SB, 0, K - 1000, 2);
    }
    if (PK >= 3000)
        return H ? make_plan_half(TB, RB, SB, TB - (PK - 3000))
                 : make_plan(TB, RB, SB, TB - (PK - 3000), TB);
    if (PK >= 2000) return H ? make_plan_half(TB, RB, SB, 0) : make_plan(TB, RB, SB, 0, TB);
    return make_plan(TB, RB, SB, 0, PK - 1000);
}

template <int TB, int RB, int PK>
__host__ __device__ constexpr bool plan_has_mf() {
    constexpr Plan P = plan_of<float, TB, RB, PK>();
    bool any = false;
    for (int j = 0; j < P.nrounds; ++j) any = any || P.r[j].mf != 0;
    return any;
}

// ---------------------------------------------------------------------------
// Split MFMA forms.  H_16 = H_2^{(x)4} applied along four tile bits is a
// 16x16 matrix of +-1 (exact in FP16 and BF16).  Each FP32 value v (pre-scaled
// by a power of two so that every |v| <= 2^14, which FP16's range needs) is
// split into hi = h(v) and lo = h(v - hi), h = fp16 (SPLIT 1) or bf16
// (SPLIT 2), both rounded to nearest (v - hi is exact in FP32), and one
// v_mfma_f32_16x16x32_{f16,bf16} computes H_16 (hi + lo) with FP32
// accumulation for a 16 x 16 block: K = 32 holds the hi and lo halves of 16
// rows.  The pair carries 22 significant bits with FP16 and 16 with BF16.
// Operand layout (lane l, i = l % 16, g = l / 16):
//   A[i][8g + j], B[8g + j][i] for j = 0..7,  D[4g + r][i] for r = 0..3.
// K order used here: k = 8g + j  ->  row 4g + (j & 3), part j >> 2 (hi, lo),
// so lane l feeds rows 4g..4g+3 and receives the same rows back.
// ---------------------------------------------------------------------------
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float f32x2c __attribute__((ext_vector_type(2)));
typedef short op8 __attribute__((ext_vector_type(8)));  // 8 halves, as bits

template <int SPLIT>
struct SplitT;
template <>
struct SplitT<1> {
    typedef _Float16 e8 __attribute__((ext_vector_type(8)));
    typedef _Float16 e2 __attribute__((ext_vector_type(2)));
    __device__ __forceinline__ static floatx4 mfma(op8 a, op8 b) {
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(e8, a),
                                                      __builtin_bit_cast(e8, b), zero, 0, 0, 0);
    }
};
template <>
struct SplitT<2> {
    typedef __bf16 e8 __attribute__((ext_vector_type(8)));
    typedef __bf16 e2 __attribute__((ext_vector_type(2)));
    __device__ __forceinline__ static floatx4 mfma(op8 a, op8 b) {
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(e8, a),
                                                       __builtin_bit_cast(e8, b), zero, 0, 0, 0);
    }
};

template <int SPLIT>
__device__ __forceinline__ op8 h16_operand() {
    using E8 = typename SplitT<SPLIT>::e8;
    using E = decltype(E8{}[0]);
    const int l = threadIdx.x & 63;
    const int i = l & 15, g = l >> 4;
    E8 a;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 4 * g + (j & 3);
        a[j] = (__builtin_popcount(i & k) & 1) ? (E)-1.0f : (E)1.0f;
    }
    return __builtin_bit_cast(op8, a);
}

// Two FP32 values to FP16 / BF16, rounded to nearest (v_cvt_pk_f16_f32,
// v_cvt_pk_bf16_f32).
template <int SPLIT>
__device__ __forceinline__ typename SplitT<SPLIT>::e2 pk_rne(float a, float b) {
    const f32x2c v = {a, b};
    return __builtin_convertvector(v, typename SplitT<SPLIT>::e2);
}

// hi/lo halves of four values in the K order above.  hi = h(v) rounded to
// nearest; v - hi is exact in FP32 (a multiple of v's FP32 ulp below 2^13 of
// them for FP16, 2^16 for BF16), and lo = h(v - hi), also rounded to nearest,
// so the split carries no systematic bias.
template <int SPLIT>
__device__ __forceinline__ op8 split4(float a, float b, float c, float d) {
    const auto hab = pk_rne<SPLIT>(a, b);
    const auto hcd = pk_rne<SPLIT>(c, d);
    const auto lab = pk_rne<SPLIT>(a - (float)hab[0], b - (float)hab[1]);
    const auto lcd = pk_rne<SPLIT>(c - (float)hcd[0], d - (float)hcd[1]);
    const typename SplitT<SPLIT>::e8 r = {hab[0], hab[1], hcd[0], hcd[1],
                                          lab[0], lab[1], lcd[0], lcd[1]};
    return __builtin_bit_cast(op8, r);
}

// One round's H_16 factor in registers.  The factor's tile bits are the
// register-index bits A, A + 1 (j) and the lane-id bits 4, 5 (g): for every
// setting q of the other register-index bits, lane 16g + c holds rows 4g + j
// of column c, which is the B operand layout, and receives rows 4g + r of the
// product in the same registers.
template <int SPLIT, int RB, int A>
__device__ __forceinline__ void mf_apply(float2 (&v)[1 << RB], const op8 amat) {
#pragma unroll
    for (int q = 0; q < (1 << (RB - 2)); ++q) {
        const int b = (q & ((1 << A) - 1)) | ((q >> A) << (A + 2));
        constexpr int s = 1 << A;
        const op8 br = split4<SPLIT>(v[b].x, v[b + s].x, v[b + 2 * s].x, v[b + 3 * s].x);
        const op8 bi = split4<SPLIT>(v[b].y, v[b + s].y, v[b + 2 * s].y, v[b + 3 * s].y);
        const floatx4 dr = SplitT<SPLIT>::mfma(amat, br);
        const floatx4 di = SplitT<SPLIT>::mfma(amat, bi);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[b + r * s] = make_float2(dr[r], di[r]);
    }
}

// The arithmetic of round J: butterflies on its FP32 bits, then its H_16
// factor (split form).
template <typename Real, int TB, int RB, int PK, int J>
__device__ __forceinline__ void round_math(typename CT<Real>::T (&v)[1 << RB], const op8 amat) {
    constexpr Round rd = plan_of<Real, TB, RB, PK>().r[J];
    butterflies<RB, rd.reg, rd.bfly>(v);
    if constexpr (rd.mf != 0) {
        static_assert(sizeof(Real) == 4, "H_16 factors act on FP32 values");
        mf_apply<PK / 10000, RB, mf_reg_index(rd)>(v, amat);
    }
}

// Rounds J .. nrounds-1 of a plan: LDS transpose, then the round's arithmetic.
template <typename Real, int TB, int RB, int PK, int J>
struct RoundRunner {
    using C = typename CT<Real>::T;
    static constexpr Plan P = plan_of<Real, TB, RB, PK>();
    static constexpr int SB = Prec<Real>::SB;
    static constexpr bool PADDED = lds_padded(P);
    static_assert(TB <= 16, "tile slots are formed for elements below 2^16");
    __device__ __forceinline__ static void run(C* lds, C (&v)[1 << RB], const op8 amat) {
        if constexpr (J < P.nrounds) {
            constexpr Round prev = P.r[J - 1];
            constexpr Round cur = P.r[J];
            if constexpr (P.half) {
                // the top tile bit is the top register-index bit of both
                // layouts: move the registers with that bit 0, then 1,
                // through half the tile's LDS (slots drop the top bit)
                constexpr uint32_t low = (1u << (TB - 1)) - 1u;
                constexpr int HR = 1 << (RB - 1);
                static_assert((prev.reg >> (TB - 1)) & (cur.reg >> (TB - 1)) & 1u, "half plan");
                __syncthreads();  // previous readers of the LDS buffer are done
                lds_put<SB, PADDED, RB - 1, prev.reg & low, prev.lperm, prev.wave, 0>(lds, v);
                __syncthreads();
                lds_get<SB, PADDED, RB - 1, cur.reg & low, cur.lperm, cur.wave, 0>(lds, v);
                __syncthreads();
                lds_put<SB, PADDED, RB - 1, prev.reg & low, prev.lperm, prev.wave, HR>(lds, v);
                __syncthreads();
                lds_get<SB, PADDED, RB - 1, cur.reg & low, cur.lperm, cur.wave, HR>(lds, v);
            } else {
                __syncthreads();  // previous readers of the LDS tile are done
                lds_put<SB, PADDED, RB, prev.reg, prev.lperm, prev.wave>(lds, v);
                __syncthreads();
                lds_get<SB, PADDED, RB, cur.reg, cur.lperm, cur.wave>(lds, v);
            }
            round_math<Real, TB, RB, PK, J>(v, amat);
            RoundRunner<Real, TB, RB, PK, J + 1>::run(lds, v, amat);
        }
    }
};

// Whole transform from round 0's register layout to the last round's.
template <typename Real, int TB, int RB, int PK>
__device__ __forceinline__ void run_transform(typename CT<Real>::T* lds,
                                              typename CT<Real>::T (&v)[1 << RB]) {
    op8 amat = {};
    if constexpr (PK >= 10000) amat = h16_operand<PK / 10000>();
    round_math<Real, TB, RB, PK, 0>(v, amat);
    RoundRunner<Real, TB, RB, PK, 1>::run(lds, v, amat);
}

// Fixed-shape tree over T doubles in LDS; segments of `seg` consecutive entries
// are reduced independently (seg divides T, both powers of two).  Result of
// segment j lands in red[j * seg].
template <int T>
__device__ __forceinline__ void seg_tree(double* red, int seg) {
    for (int s = seg >> 1; s >= 1; s >>= 1) {
        __syncthreads();
        const int i = threadIdx.x;
        if ((i & (2 * s - 1)) < s) red[i] += red[i + s];
    }
    __syncthreads();
}

}  // namespace sre2
