// sre2_half.hip - on-chip half transforms: S_x of whole shifts, 10 <= N <= 16
// (FP32) / 15 (FP64), for every form but the BF16 split one (FP16: from 13 on).
//
// For x != 0, f_x(k ^ x) = conj f_x(k) (the summand of Eq. 3 at k and k ^ x),
// so with hb a set bit of x the transform A of f_x over the half space
// k_hb = 0 holds every Pauli expectation of the shift: W_x(z) is 2 Re A or
// 2i Im A, and S_x = 16 sum (Re^4 + Im^4).  Shift 0 has no such pairing, but
// f_0 = |psi|^2 is real: the two halves k_hb = 0 and 1 are carried as the real
// and imaginary part of one complex transform, and one last stage A.re +- A.im
// gives W_0.  Its bits are assigned so that its stages run in the order of the
// plain transform of 2^N values, and W_0, a quarter of a Haar state's S, keeps
// its bits.
//
// A workgroup holds one half transform of 2^(N-1) complex values in registers
// and transposes it between rounds through an LDS buffer of one real part
// (2^(N-1) floats or doubles), first the real parts, then the imaginary ones.
// That buffer is what sets the occupancy: at N = 14 a complex buffer leaves
// two workgroups (2 waves per SIMD) on a CU and a real one four, and the
// kernel takes 163 us instead of 193 (the full transforms of k_fused, which
// it replaces: 450 us); the same buffer lets N = 15 and 16 (FP64: 14 and 15)
// stay on chip at all, where the two passes through HBM moved 8 (16) bytes
// per Pauli string (N = 16 FP32: 6.9 ms before, 4.2 ms here; FP64 N = 15:
// 3.2 ms before, 1.55 ms).  The bound is the VALU: N - 1 additions, the
// product (2) and the term (3) per Pauli string, 0.13 ms at N = 14.
//
// Measured and not taken (N = 14 FP32): keeping psi[k] and psi[k ^ x] in
// registers over 8 or 32 shifts that differ in register bits only (no loads
// after the first; two waves per SIMD for the registers): 170-176 us; 16
// values per thread instead of 32: 174 us.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_half_map.h"
#include "sre2_tile.h"

namespace sre2 {

namespace {

// conj(a) * b, both parts fused (no identity between f_x(k) and f_x(k ^ x)
// is needed here).
template <typename C>
__device__ __forceinline__ C cmul_conj_f(C a, C b) {
    C r;
    r.x = a.x * b.x + a.y * b.y;
    r.y = a.x * b.y - a.y * b.x;
    return r;
}

// One part (0: re, 1: im) of the registers to (PUT) or from a padded buffer
// of reals.  Slots are 4 or 8 bytes: with pad<5> 32 consecutive lanes hit 32
// distinct slots modulo 32, free of conflicts for both (two lanes share a slot in the
// last round of N = 10 and 11, which have too few bits to choose from).  ds_read /
// ds_write offsets are 16 bits: slots above kLdsSplit bytes take a second base,
// which covers 96 KiB; beyond (the upper slots of the 132 KiB buffers of N = 16
// in FP32, 15 in FP64) the compiler adds to the address.
constexpr uint32_t kLdsSplit = 32768;
template <bool PUT, int PART, int RB, uint32_t REG, uint32_t LPERM, uint32_t WAVE, typename Real,
          typename C>
__device__ __forceinline__ void lds_part(Real* lds, C (&v)[1 << RB]) {
    constexpr int SB = kHalfSB;
    char* b = reinterpret_cast<char*>(lds) +
              pad16<SB>(thread_base<LPERM, WAVE>()) * (uint32_t)sizeof(Real);
    char* b2 = b + kLdsSplit;
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) {
        const uint32_t off = pad<SB>(pdep((uint32_t)i, REG)) * (uint32_t)sizeof(Real);
        Real* p = reinterpret_cast<Real*>(off >= kLdsSplit ? b2 + (off - kLdsSplit) : b + off);
        if constexpr (PUT)
            *p = PART ? v[i].y : v[i].x;
        else
            (PART ? v[i].y : v[i].x) = *p;
    }
}

// Rounds J .. nrounds - 1 of the half transform.
template <typename Real, int NT, int RB, int SPLIT, int J>
struct HalfRunner {
    using C = typename CT<Real>::T;
    static constexpr Plan P = half_plan<NT, RB, SPLIT>();
    static constexpr int NV = half_lds_reals(P);
    __device__ __forceinline__ static void math(C (&v)[1 << RB], const op8 amat) {
        constexpr Round c = P.r[J];
        butterflies<RB, c.reg, c.bfly>(v);
        if constexpr (c.mf != 0) mf_apply<SPLIT, RB, mf_reg_index(c)>(v, amat);
    }
    __device__ __forceinline__ static void run(Real* lds, C (&v)[1 << RB], const op8 amat) {
        if constexpr (J < P.nrounds) {
            constexpr Round a = P.r[J - 1];
            constexpr Round c = P.r[J];
            __syncthreads();  // previous readers of the buffer are done
            lds_part<true, 0, RB, a.reg, a.lperm, a.wave>(lds, v);
            __syncthreads();
            lds_part<false, 0, RB, c.reg, c.lperm, c.wave>(lds, v);
            __syncthreads();
            lds_part<true, 1, RB, a.reg, a.lperm, a.wave>(lds, v);
            __syncthreads();
            lds_part<false, 1, RB, c.reg, c.lperm, c.wave>(lds, v);
            math(v, amat);
            HalfRunner<Real, NT, RB, SPLIT, J + 1>::run(lds, v, amat);
        }
    }
};

// Waves per SIMD asked of the compiler: with 64 registers of values per thread
// four fit (128 registers each), with 128 (FP64 N = 14, 15) two.
// (The histogram's terms spill a few words at four; three waves without spills
// are slower: 163 against 151 us at N = 13 FP32.)
template <typename Real>
__host__ __device__ constexpr int half_waves_per_simd(int rb) {
    return (1 << rb) * (int)sizeof(Real) > 128 ? 2 : 4;
}

// Blocks of a histogram launch: each adds its bins to the global counters once
// (one block per shift would queue 2^N of them at the same few addresses), and
// takes four shifts or more.
constexpr int64_t kHistBlocks = 2048;

// Reductions: the sum of |W|^4, the general sums, the histogram.
enum HalfRed { RED_QUARTIC, RED_GEN, RED_HIST };

// Block b of the grid takes shift x_begin + b, and with RED_HIST every
// gridDim.x-th one from there (so that few blocks add to the global counters).
// SPLIT (1): shifts x >= 1 of the FP16 split form, values scaled by
// 2^*scale_exp; N = 14 442 -> 156 us, N = 16 10.0 -> 4.3 ms.  Shift 0, whose W_0
// is a quarter of S, keeps the order of its matrix products: the other kernels
// of the form take it.  The BF16 form is not taken here: under another order its
// 16-bit halves move the S_x of N = 13 to 16 by 2e-9 to 1.5e-8 (2-norm), FP16's
// 22 bits by 4e-10 or less.
template <typename Real, int NT, int RB, int RED, int SPLIT, typename PackT>
__global__ __launch_bounds__(1 << (NT - RB))
__attribute__((amdgpu_waves_per_eu(half_waves_per_simd<Real>(RB))))
void k_half(const typename CT<Real>::T* __restrict__ psi, int64_t x_begin, int64_t x_count,
            double* __restrict__ S_out, const int* __restrict__ scale_exp, const PackT pk,
            const Spec sp, int bit) {
    static_assert(!SPLIT || (RED == RED_QUARTIC && sizeof(Real) == 4), "split forms: M2 in FP32");
    using C = typename CT<Real>::T;
    using HR = HalfRunner<Real, NT, RB, SPLIT, 1>;
    constexpr int N = NT + 1;
    constexpr int NW = (1 << (NT - RB)) / 64;
    constexpr int NE = 1 << RB;
    constexpr Round r0 = HR::P.r[0];
    static_assert(RED != RED_HIST || sizeof(Real) == 8 || RB == 5, "HB_LAST's stage order");
    __shared__ Real lds[HR::NV];
    __shared__ double red[NW];
    __shared__ unsigned lh[RED == RED_HIST ? kMaxBins * kHistCopies : 1];
    if constexpr (is_packed<PackT>) {
        psi = (const C*)pk.psi[blockIdx.y];
        S_out = pk_sx(pk.ws[blockIdx.y], N) + x_begin;
        scale_exp = pk_se(pk.ws[blockIdx.y], N);
    }
    const int se = SPLIT ? *scale_exp : 0;
    op8 amat = {};
    if constexpr (SPLIT != 0) amat = h16_operand<SPLIT>();
    Real lnorm2 = Real(0);
    if constexpr (RED == RED_HIST) {
        hist_clear(lh, sp);
        lnorm2 = hist_lnorm2<Real>(sp);
    }
    const auto rs = buf_rsrc(psi, (uint32_t)sizeof(C) << N);
    const uint32_t base = thread_base<r0.lperm, r0.wave>();
    const auto one_shift = [&](uint32_t at) {
        const uint32_t x = (uint32_t)x_begin + at;
        const bool zero = SPLIT == 0 && x == 0;
        C v[NE];
        if (zero) {
            // a rolled loop through the thread's own LDS slots, so that one
            // workgroup's case does not cost the others registers
            static_assert(SPLIT || r0.reg == top_bits(bits_range(0, NT), RB), "element bits");
            constexpr BitOrder map = zero_map<Real, NT, RB>();
            const auto squares = [&](uint32_t half) {
#pragma unroll 1
                for (uint32_t i = 0; i < NE; ++i) {
                    const uint32_t e = base | (i << (NT - RB));
                    uint32_t q = half << map.bit[NT];
#pragma unroll
                    for (int b = 0; b < NT; ++b) q |= ((e >> b) & 1u) << map.bit[b];
                    const C c = load_at<C>(rs, q, 0);
                    lds[pad16<kHalfSB>(e)] = cmul_conj_a(c, c).x;
                }
            };
            squares(0u);
            lds_part<false, 0, RB, r0.reg, r0.lperm, r0.wave>(lds, v);
            squares(1u);
            lds_part<false, 1, RB, r0.reg, r0.lperm, r0.wave>(lds, v);
        } else {
            // element e -> k, the map putting a zero at bit hb, and the partner
            // k ^ x; both act on disjoint bits of the thread's and the
            // register's part of e, so the register's part of an address is
            // uniform (a scalar offset)
            constexpr bool HIST = RED == RED_HIST;
            const HalfShift hs = half_shift<HIST>(x, N, bit);
            const auto k_of = [&](uint32_t e) { return half_k<HIST>(e, N, hs); };
            const uint32_t R = k_of(r0.reg);
            const uint32_t kb = k_of(base);
            const uint32_t vb = kb ^ (x & ~R), xr = x & R;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const uint32_t kr = k_of(pdep((uint32_t)i, r0.reg));
                if constexpr (RED == RED_HIST)
                    v[i] = cmul_conj_a(load_at<C>(rs, vb, kr ^ xr), load_at<C>(rs, kb, kr));
                else
                    v[i] = cmul_conj_f(load_at<C>(rs, vb, kr ^ xr), load_at<C>(rs, kb, kr));
            }
            if constexpr (SPLIT != 0) {
                const Real sc = ldexpf(1.0f, se);
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    v[i].x *= sc;
                    v[i].y *= sc;
                }
            }
        }
        HalfRunner<Real, NT, RB, SPLIT, 0>::math(v, amat);
        HR::run(lds, v, amat);
        double acc = 0.0;
        if (zero) {
            // the last stage, across the two halves: two values of W, halved
            // (exactly) to go through the same sum as 2 Re and 2 Im
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const Real a = v[i].x + v[i].y, c = v[i].x - v[i].y;
                v[i].x = Real(0.5) * a;
                v[i].y = Real(0.5) * c;
            }
        }
        if constexpr (RED == RED_QUARTIC) {
#pragma unroll
            for (int i = 0; i < NE; ++i) acc += abs4h(v[i]);
            acc *= SPLIT ? ldexp(16.0, -4 * se) : 16.0;
        } else {
            acc = gen_sum<Real, GEN_HERM, RED == RED_HIST>(v, sp, lnorm2, lh);
        }
        if constexpr (RED == RED_HIST) {  // its sum is 0 in every shift
            if (threadIdx.x == 0) S_out[at] = acc;
            return;
        }
        acc = wave_sum(acc);
        if constexpr (NW == 1) {
            if (threadIdx.x == 0) S_out[at] = acc;
        } else {
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
            __syncthreads();
            if (threadIdx.x == 0) {
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) t += red[w];
                S_out[at] = t;
            }
        }
    };
    if constexpr (RED == RED_HIST) {
        for (uint32_t at = blockIdx.x; at < (uint32_t)x_count; at += gridDim.x) {
            __syncthreads();  // the previous shift's readers of the buffer
            one_shift(at);
        }
        hist_flush(lh, sp);
    } else {
        one_shift(blockIdx.x);
    }
}

template <typename Real, int N, int RED, int SPLIT>
hipError_t launch_half_n(const void* psi, int64_t x0, int64_t xc, double* S, const int* se,
                         const Pack& pk, const Spec& sp, int bit, hipStream_t st) {
    using C = typename CT<Real>::T;
    constexpr int RB = half_rb<Real>(N, RED == RED_HIST || SPLIT);
    const int64_t blocks =
        RED != RED_HIST ? xc : ((xc + 3) / 4 < kHistBlocks ? (xc + 3) / 4 : kHistBlocks);
    const dim3 block(1 << (N - 1 - RB));
    if constexpr (RED == RED_QUARTIC && N <= Tune<Real>::FMAX) {
        if (pk.count) {
            k_half<Real, N - 1, RB, RED, SPLIT, Pack>
                <<<dim3((unsigned)blocks, (unsigned)pk.count), block, 0, st>>>(
                    (const C*)psi, x0, xc, S, se, pk, sp, bit);
            return hipGetLastError();
        }
    }
    if (pk.count) return hipErrorInvalidValue;
    k_half<Real, N - 1, RB, RED, SPLIT, NoPack><<<dim3((unsigned)blocks), block, 0, st>>>(
        (const C*)psi, x0, xc, S, se, NoPack{}, sp, bit);
    return hipGetLastError();
}

template <typename Real, int RED, int SPLIT, int... Ns>
hipError_t dispatch_half(int N, const void* psi, int64_t x0, int64_t xc, double* S, const int* se,
                         const Pack& pk, const Spec& sp, int bit, hipStream_t st,
                         std::integer_sequence<int, Ns...>) {
    hipError_t e = hipErrorInvalidValue;
    constexpr int N0 = SPLIT             ? Tune<Real>::HSPLIT
                       : RED == RED_HIST ? half_hist_min<Real>()
                                         : Tune<Real>::HMIN;
    ((N == Ns + N0
          ? (e = launch_half_n<Real, Ns + N0, RED, SPLIT>(psi, x0, xc, S, se, pk, sp, bit, st), 0)
          : 0),
     ...);
    return e;
}

}  // namespace

template <typename Real>
hipError_t launch_half(const void* psi, int N, bool herm, int split, int64_t x0, int64_t xc,
                       double* S, const int* se, const Pack& pk, const Spec* sp, hipStream_t st) {
    using T = Tune<Real>;
    const bool hist = sp && sp->kind == kRedHist;
    if (xc < 1 || x0 < (split ? 1 : 0) || x0 + xc > ((int64_t)1 << N)) return hipErrorInvalidValue;
    constexpr auto ns = std::make_integer_sequence<int, T::HMAX - T::HMIN + 1>{};
    constexpr auto hs =
        std::make_integer_sequence<int, half_hist_max<Real>() - half_hist_min<Real>() + 1>{};
    const Spec none{};
    if constexpr (sizeof(Real) == 4) {
        constexpr auto ss = std::make_integer_sequence<int, T::HMAX - T::HSPLIT + 1>{};
        if (split && sp) return hipErrorInvalidValue;
        if (split == 1)
            return dispatch_half<Real, RED_QUARTIC, 1>(N, psi, x0, xc, S, se, pk, none, HB_TOP, st,
                                                       ss);
    }
    if (split) return hipErrorInvalidValue;
    if (hist)
        return dispatch_half<Real, RED_HIST, 0>(N, psi, x0, xc, S, se, pk, *sp,
                                                herm || sizeof(Real) == 8 ? HB_TOP : HB_LAST, st,
                                                hs);
    if (sp) return dispatch_half<Real, RED_GEN, 0>(N, psi, x0, xc, S, se, pk, *sp, HB_TOP, st, ns);
    return dispatch_half<Real, RED_QUARTIC, 0>(N, psi, x0, xc, S, se, pk, none, HB_TOP, st, ns);
}
template hipError_t launch_half<float>(const void*, int, bool, int, int64_t, int64_t, double*,
                                       const int*, const Pack&, const Spec*, hipStream_t);
template hipError_t launch_half<double>(const void*, int, bool, int, int64_t, int64_t, double*,
                                        const int*, const Pack&, const Spec*, hipStream_t);

}  // namespace sre2
