// sre2_pass2.hip - pass 2 of the two-pass transforms (columns, terms of the
// Pauli sums), and where the row pairs start.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_both.h"
#include "sre2_twopass.h"

namespace sre2 {

// ---------------------------------------------------------------------------
// Two-pass, pass 2: column transform over the HT row bits of one shift's slab
// (2^NS values = 2^HT rows of 2^L).  A tile is 2^HT rows x 2^(TB-HT) columns.
// Block b -> shift slot b / P, column group b % P; the group loops over its
// column tiles and writes one FP64 partial of S_x.
//  HALF_NONE  a full slab: sum of |W|^4.
//  HALF_SLAB  a half slab (Hermitian pair, row pairs: the rows with bit
//             j = half_row_bit(x >> L) clear).  With xh = x >> L and
//             xl = x mod 2^L, f_x(k ^ x) = conj f_x(k) makes the left-out row
//               row(r ^ xh)[z] = (-1)^popcount(z & xl) conj(row(r)[z]),
//             so with A the column transform of the stored rows the last
//             stage, along j, would give A +- conj A: W is 2 Re A and 2i Im A,
//             and S_x = 16 sum (Re^4 + Im^4).
//  HALF_BOTH  a full slab with that same order of stages (row pairs switched
//             off): the rows with bit j clear and set are transformed apart
//             and combined last, sum of |W|^4 over both of the combined values
//             (both_terms).  Row identity and column transform hold bit for bit
//             in the plain forms: the products are exactly conjugate
//             (cmul_conj_a), and a butterfly network fed an XOR-permuted input
//             computes the same sums and differences, some of them negated
//             (u + v = v + u, v - u = -(u - v)); so the combined values are
//             exactly (2 Re A, 0) and (0, 2 Im A), and S_x has every bit of the
//             half slab's - from all rows of the slab, and only if they hold
//             the pairing.
// (The split forms' H_16 products on the matrix cores sum in an order the
// permutation does not preserve: their half slabs hold the exact images of
// the computed stored rows, equal to the full slab's up to rounding.)
//
// What bounds it: reading the slab (FP32 half slabs at N = 20: 16 GiB per
// 4096-shift launch in 2.4 ms, 7.1 TB/s).  The row pairs first rebuilt the
// left-out rows by sign flips and ran the full column transform (3.9 ms, bound
// by its arithmetic: 8 instead of 7 stages on twice the values); at N = 22 and
// 24 that took 128 KiB half-LDS tiles, where the stored rows alone fit 64 KiB.
// ---------------------------------------------------------------------------
enum HalfMode { HALF_NONE, HALF_SLAB, HALF_BOTH };

template <typename Real, int HT, int TB, int RB, int HALF, int SPLIT, bool GEN>
__global__ __launch_bounds__(1 << (TB - RB))
__attribute__((amdgpu_waves_per_eu(half_lds<Real>(TB) ? half_waves(TB, RB)
                                   : (SPLIT ? SRE2_P2S_WAVES : SRE2_P2_WAVES))))
void k_pass2(const typename CT<Real>::T* __restrict__ scratch, int NS, int P,
             double* __restrict__ part, const int* __restrict__ scale_exp, const Spec sp,
             int64_t x0) {
    static_assert(HALF != HALF_BOTH || (!SPLIT && !GEN), "comparison path of the plain M2 forms");
    using C = typename CT<Real>::T;
    constexpr int T = 1 << (TB - RB);
    constexpr int PK = 3000 + HT + 10000 * SPLIT;
    constexpr Plan PL = plan_of<Real, TB, RB, PK>();
    constexpr Round r0 = PL.r[0];
    constexpr int CB = TB - HT;  // column bits per tile
    constexpr uint32_t CMASK = (1u << CB) - 1u;
    // streaming loads only when a tile reads whole 128-byte lines of a row
    constexpr bool NT = SRE2_NT_SLAB && ((int)sizeof(C) << CB) >= 128;
    __shared__ C lds[lds_values(PL)];
    __shared__ double red[T];
    __shared__ unsigned lh[GEN ? kMaxBins * kHistCopies : 1];
    Real lnorm2 = Real(0);
    if constexpr (GEN) {
        hist_clear(lh, sp);
        lnorm2 = hist_lnorm2<Real>(sp);
    }

    const int64_t b = blockIdx.x;
    const int64_t s = b / P;
    const int g = (int)(b % P);
    // bits of one shift's slab; row bits of pass 1 (HALF_BOTH transforms the
    // HT + 1 row bits of its full slab in two halves)
    const int L = NS - HT - (HALF == HALF_BOTH ? 1 : 0);
    const int ntile = 1 << (L - CB);  // column tiles per shift
    const int per = ntile / P;
    const auto rs = buf_rsrc(scratch + ((uint64_t)s << NS), (uint32_t)sizeof(C) << NS);
    // tile element e -> slab offset (e >> CB) * 2^L + (e & CMASK), which adds
    // over disjoint bits: the thread's part once, the register element's part
    // (and the column tile's) as a uniform offset.  HALF_BOTH: the row with
    // a zero inserted at bit j, which keeps bits disjoint.
    const uint32_t base = thread_base<r0.lperm, r0.wave>();
    int j = 0;
    if constexpr (HALF == HALF_BOTH) j = half_row_bit((uint32_t)((uint64_t)(x0 + s) >> L), 0u);
    const auto row_of = [&](uint32_t r) { return HALF == HALF_BOTH ? insert0(r, (uint32_t)j) : r; };
    const uint32_t vb = (row_of(base >> CB) << L) + (base & CMASK);
    double acc = 0.0;
    const auto load_tile = [&](C (&v)[1 << RB], int ct, uint32_t half) {
        const uint32_t cto = ((uint32_t)ct << CB) + (half << (j + L));
#pragma unroll
        for (int i = 0; i < (1 << RB); ++i) {
            const uint32_t r = pdep((uint32_t)i, r0.reg);
            v[i] = load_at<C, NT ? 2 : 0>(rs, vb, cto + (row_of(r >> CB) << L) + (r & CMASK));
        }
    };
    // column transform of one tile and its terms, tiles in ascending order
    const auto consume = [&](C (&v)[1 << RB]) {
        run_transform<Real, TB, RB, PK>(lds, v);
        if constexpr (GEN) {
            acc += gen_sum<Real, HALF == HALF_SLAB ? GEN_HERM : GEN_PLAIN, true>(v, sp, lnorm2, lh);
        } else {
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i)
                acc += HALF == HALF_SLAB ? abs4h(v[i]) : abs4(v[i]);
        }
    };
    const int c0 = g * per, c1 = (g + 1) * per;
    // Tiles that fit the LDS whole load the next tile while transforming this
    // one (two register sets; these kernels are held to two waves per SIMD by
    // their LDS tiles, which leaves the registers; the full-slab split kernel
    // and split tiles above 2^12 values have none to spare); barriers wait on
    // LDS only, so the loads stay in flight across the transform.
    constexpr bool PREFETCH =
        !half_lds<Real>(TB) && (!SPLIT || (HALF == HALF_SLAB && TB <= 12)) && !GEN;
    if constexpr (HALF == HALF_BOTH) {
        constexpr Round rl = PL.r[PL.nrounds - 1];
        const uint64_t x = (uint64_t)(x0 + s);
        const uint32_t xl = (uint32_t)x & ((1u << L) - 1u);
        const uint32_t xt = both_mask((uint32_t)(x >> L), xl, j, CB);
        const uint32_t odd_t = parity(thread_base<rl.lperm, rl.wave>() & xt);
        for (int ct = c0; ct < c1; ++ct) {
            C v[1 << RB], u[1 << RB];
            load_tile(v, ct, 0);
            load_tile(u, ct, 1);
            run_transform<Real, TB, RB, PK>(lds, v);
            run_transform<Real, TB, RB, PK>(lds, u);
            const uint32_t odd = odd_t ^ parity(((uint32_t)ct << CB) & xl);
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i)
                acc += both_terms(v[i], u[i], odd ^ parity(pdep((uint32_t)i, rl.reg) & xt));
        }
    } else if constexpr (PREFETCH) {
        C va[1 << RB], vn[1 << RB];
        load_tile(va, c0, 0);
        for (int ct = c0; ct < c1; ct += 2) {
            if (ct + 1 < c1) load_tile(vn, ct + 1, 0);
            consume(va);
            if (ct + 1 < c1) {
                if (ct + 2 < c1) load_tile(va, ct + 2, 0);
                consume(vn);
            }
        }
    } else {
        for (int ct = c0; ct < c1; ++ct) {
            C v[1 << RB];
            load_tile(v, ct, 0);
            consume(v);
        }
    }
    if constexpr (!GEN) {
        if constexpr (HALF == HALF_SLAB) acc *= 16.0;
        if constexpr (SPLIT) acc *= ldexp(1.0, -4 * *scale_exp);
    }
    const double tot = block_sum<T>(acc, red);
    if (threadIdx.x == 0) part[b] = tot;
    if constexpr (GEN) hist_flush(lh, sp);
}

namespace {

template <typename Real, int HT, int HALF, int SPLIT, bool GEN>
hipError_t launch_pass2_ht(const void* scratch, int NS, int cs, int P, double* part, const int* se,
                           const Spec& sp, int64_t x0, hipStream_t st) {
    using C = typename CT<Real>::T;
    constexpr int TB = pass2_tb<Real>(HT), RB = Tune<Real>::RB2;
    hipLaunchKernelGGL((k_pass2<Real, HT, TB, RB, HALF, SPLIT, GEN>),
                       dim3((unsigned)((int64_t)cs * P)), dim3(1 << (TB - RB)), 0, st,
                       (const C*)scratch, NS, P, part, se, sp, x0);
    return hipGetLastError();
}

// Row bits of the smallest size that takes two passes: N = HMAX + 1 (the FP32
// histogram from half_hist_max + 1, the split forms' full slabs from FMAX + 1, for
// shift 0 at least; BF16 half slabs from kImagesMaxN + 1).
template <typename Real, int HALF, int SPLIT, bool GEN>
constexpr int pass2_min_rows() {
    using T = Tune<Real>;
    int N = T::HMAX + 1;
    if (GEN) N = half_hist_max<Real>() + 1;
    if (SPLIT) N = HALF == HALF_NONE ? T::FMAX + 1 : SPLIT == 2 ? kImagesMaxN + 1 : T::HMAX + 1;
    return N - T::ROW - (HALF == HALF_NONE ? 0 : 1);
}

template <typename Real, int HALF, int SPLIT, bool GEN, int... Hs>
hipError_t dispatch_pass2_of(int HT, const void* scratch, int NS, int cs, int P, double* part,
                             const int* se, const Spec& sp, int64_t x0, hipStream_t st,
                             std::integer_sequence<int, Hs...>) {
    constexpr int H0 = pass2_min_rows<Real, HALF, SPLIT, GEN>();
    hipError_t e = hipErrorInvalidValue;
    ((HT == Hs + H0 ? (e = launch_pass2_ht<Real, Hs + H0, HALF, SPLIT, GEN>(
                           scratch, NS, cs, P, part, se, sp, x0, st),
                       0)
                    : 0),
     ...);
    return e;
}
template <typename Real, int HALF, int SPLIT, bool GEN>
hipError_t dispatch_pass2(int HT, const void* scratch, int NS, int cs, int P, double* part,
                          const int* se, const Spec& sp, int64_t x0, hipStream_t st) {
    constexpr int n = pass2_max_rows<Real>() - pass2_min_rows<Real, HALF, SPLIT, GEN>() + 1;
    return dispatch_pass2_of<Real, HALF, SPLIT, GEN>(HT, scratch, NS, cs, P, part, se, sp, x0, st,
                                                     std::make_integer_sequence<int, n>{});
}

}  // namespace

// First shift of the row-pair range of an N-qubit evaluation (split form
// `split`): 2^L, or in the plain forms 2^(L + r) where the column transform of
// a full slab needs a tile above 64 KiB, r the lowest register row bit of that
// tile's plan.
template <typename Real>
int64_t pair_first_shift(int N, int split) {
    if (N <= Tune<Real>::FMAX || N > max_n_of<Real>()) return (int64_t)1 << N;
    const int L = row_bits_of<Real>(N), HT = N - L;
    const int tb = pass2_tb<Real>(HT);
    if (split || !half_lds<Real>(tb)) return (int64_t)1 << L;
    const Plan p = make_plan_half(tb, Tune<Real>::RB2, Prec<Real>::SB, tb - HT);
    return (int64_t)1 << (L + __builtin_ctz(p.r[0].reg >> (tb - HT)));
}
template int64_t pair_first_shift<float>(int, int);
template int64_t pair_first_shift<double>(int, int);

template <typename Real>
hipError_t launch_pass2(const void* scratch, int N, int slab, int split, int64_t x0, int cs,
                        int P, double* part, const int* se, const Spec* sp, hipStream_t st) {
    if (N <= Tune<Real>::FMAX || N > max_n_of<Real>()) return hipErrorInvalidValue;
    if (slab < kSlabFull || slab > kSlabImages || split < 0 || split > 2 ||
        (split && (slab == kSlabHerm || sizeof(Real) != 4)) ||
        (slab == kSlabBoth && (sp || split)) ||
        (slab == kSlabImages && (sp || split != 2 || N > kImagesMaxN)))
        return hipErrorInvalidValue;
    int NS, L;
    slab_geometry<Real>(N, slab, &NS, &L);
    if (slab != kSlabFull && slab != kSlabHerm && x0 < pair_first_shift<Real>(N, split))
        return hipErrorInvalidValue;
    if (slab == kSlabImages) return launch_pass2_images(scratch, N, x0, cs, P, part, se, st);
    const bool half = slab == kSlabHerm || slab == kSlabPairs;
    const int HT = NS - L - (slab == kSlabBoth ? 1 : 0);
    if (sp) {
        if (split || sp->kind < kRedPow || sp->kind > kRedHist ||
            (sp->kind == kRedHist && (!sp->hist || !sp->nrm || sp->nbins < 2 ||
                                      sp->nbins > kMaxBins)))
            return hipErrorInvalidValue;
        if (half)
            return dispatch_pass2<Real, HALF_SLAB, 0, true>(HT, scratch, NS, cs, P, part, se, *sp,
                                                            x0, st);
        return dispatch_pass2<Real, HALF_NONE, 0, true>(HT, scratch, NS, cs, P, part, se, *sp, x0,
                                                        st);
    }
    const Spec none{};
    if constexpr (sizeof(Real) == 4) {
        if (split == 1)
            return half ? dispatch_pass2<Real, HALF_SLAB, 1, false>(HT, scratch, NS, cs, P, part,
                                                                    se, none, x0, st)
                        : dispatch_pass2<Real, HALF_NONE, 1, false>(HT, scratch, NS, cs, P, part,
                                                                    se, none, x0, st);
        if (split == 2)
            return half ? dispatch_pass2<Real, HALF_SLAB, 2, false>(HT, scratch, NS, cs, P, part,
                                                                    se, none, x0, st)
                        : dispatch_pass2<Real, HALF_NONE, 2, false>(HT, scratch, NS, cs, P, part,
                                                                    se, none, x0, st);
    }
    if (half)
        return dispatch_pass2<Real, HALF_SLAB, 0, false>(HT, scratch, NS, cs, P, part, se, none,
                                                         x0, st);
    if (slab == kSlabBoth)
        return dispatch_pass2<Real, HALF_BOTH, 0, false>(HT, scratch, NS, cs, P, part, se, none,
                                                         x0, st);
    return dispatch_pass2<Real, HALF_NONE, 0, false>(HT, scratch, NS, cs, P, part, se, none, x0,
                                                     st);
}

template hipError_t launch_pass2<float>(const void*, int, int, int, int64_t, int, int, double*,
                                        const int*, const Spec*, hipStream_t);
template hipError_t launch_pass2<double>(const void*, int, int, int, int64_t, int, int, double*,
                                         const int*, const Spec*, hipStream_t);

}  // namespace sre2
