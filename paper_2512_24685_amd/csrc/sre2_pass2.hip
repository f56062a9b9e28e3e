// sre2_pass2.hip - pass 2 of the two-pass transforms (columns, terms of the
// Pauli sums), and where the row pairs start.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_twopass.h"

namespace sre2 {

// ---------------------------------------------------------------------------
// Row pairs (plain and split forms, shifts x >= 2^L).  With xh = x >> L and
// xl = x mod 2^L, f_x(k ^ x) = conj f_x(k) makes slab row r ^ xh of pass 1
// the row r transformed with its input XOR-permuted by xl and conjugated, so
//   row(r ^ xh)[z] = (-1)^popcount(z & xl) conj(row(r)[z]).
// That holds bit for bit: the products are exactly conjugate (cmul_conj_a),
// and a butterfly network fed an XOR-permuted input computes the same sums
// and differences, some of them negated (u + v = v + u, v - u = -(u - v)).
// So pass 1 stores only the rows with bit j = half_row_bit(xh, register row
// bits of the pass-2 tile) clear, and pass 2 rebuilds a row with bit j set
// from its partner: conjugate and sign are sign-bit flips, and the column
// transform then runs on exactly the values of the full slab.  (The split
// forms' H_16 products on the matrix cores sum in an order the permutation
// does not preserve: there the rebuilt rows are the exact images of the
// computed stored rows, equal to the full slab's up to rounding.)  A launch
// covers shifts of one row part xh (its chunk stays inside one block of 2^L
// shifts), so j is one value per launch and the kernel runs a tile loop
// specialised on it: j is taken among the register row bits when xh has one,
// so that which elements are rebuilt is fixed per register index
// (pair_load_reg); otherwise xh has only thread row bits and whole threads
// hold rebuilt rows (pair_load_thr; not in the plain half-LDS tiles, whose
// row pairs start where xh has a register row bit, pair_first_shift, and
// which form the thread's address parts per tile to stay within their
// registers).  Stored values are read twice (as
// themselves and as a partner) inside one tile, the second time from the
// caches.
// ---------------------------------------------------------------------------
template <typename C, int RB, uint32_t REG, int CB, int J>
__device__ __forceinline__ void pair_load_reg(C (&v)[1 << RB], __amdgpu_buffer_rsrc_t rs, int L,
                                              uint32_t vb0, uint32_t vb1, uint32_t xh,
                                              uint32_t xl, uint32_t cto, uint32_t mT) {
    constexpr uint32_t CMASK = (1u << CB) - 1u;
    const uint32_t xhr = xh & (REG >> CB);  // xh on the register row bits
    // conjugate: the imaginary part flips; the empty asm keeps the compiler
    // from splitting y ^ mTy back into two XORs per element
    uint32_t mTy = mT ^ kSign;
    asm volatile("" : "+v"(mTy));
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) {
        const uint32_t r = pdep((uint32_t)i, REG);
        const uint32_t R = r >> CB, cr = r & CMASK;
        if ((R >> J) & 1u) {  // a rebuilt row: partner row ^ xh, stored
            const uint32_t sr = cr ? ((__builtin_popcount(cr & xl) & 1u) ? kSign : 0u) : 0u;
            const C t = load_at<C>(rs, vb1, (remove_bit(R ^ xhr, J) << L) + cto + cr);
            v[i] = xor_signs(t, mT ^ sr, mTy ^ sr);
        } else {
            v[i] = load_at<C>(rs, vb0, (remove_bit(R, J) << L) + cto + cr);
        }
    }
}

// Calls f(std::integral_constant<int, j>) for the register row bit j.
template <uint32_t RROW, int JJ = 0, typename F>
__device__ __forceinline__ void with_reg_row_bit(int j, F&& f) {
    if constexpr (JJ < 32) {
        if constexpr ((RROW >> JJ) & 1u) {
            if (j == JJ) {
                f(std::integral_constant<int, JJ>{});
                return;
            }
        }
        with_reg_row_bit<RROW, JJ + 1>(j, f);
    }
}

// j a thread row bit (xh has no register row bit): a thread's rows are all
// stored (fm = 0) or all rebuilt (fm = ~0); vb already points at the stored rows.
template <typename C, int RB, uint32_t REG, int CB>
__device__ __forceinline__ void pair_load_thr(int j, C (&v)[1 << RB], __amdgpu_buffer_rsrc_t rs,
                                              int L, uint32_t vb, uint32_t fm, uint32_t xl,
                                              uint32_t cto, uint32_t mT) {
    constexpr uint32_t CMASK = (1u << CB) - 1u;
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) {
        const uint32_t r = pdep((uint32_t)i, REG);
        const uint32_t R = r >> CB, cr = r & CMASK;
        const uint32_t m = fm & (mT ^ ((__builtin_popcount(cr & xl) & 1u) ? kSign : 0u));
        const C t = load_at<C>(rs, vb, (remove_bit(R, j) << L) + cto + cr);
        v[i] = xor_signs(t, m, m ^ (fm & kSign));
    }
}

// ---------------------------------------------------------------------------
// Two-pass, pass 2: column transform over the HT slab-row bits of one shift's
// slab (2^NS values = 2^HT rows of 2^L; with PAIR the slab holds the 2^(HT-1)
// stored rows of the row pairs, and x0 is the chunk's first shift).  A tile
// is 2^HT rows x 2^(TB-HT) columns.  Block b -> shift slot b / P, column
// group b % P; the group loops over its column tiles and writes one FP64
// partial of S_x.
// ---------------------------------------------------------------------------
template <typename Real, int HT, int TB, int RB, bool HERM, int SPLIT, bool GEN, bool PAIR>
__global__ __launch_bounds__(1 << (TB - RB))
__attribute__((amdgpu_waves_per_eu(half_lds<Real>(TB) ? half_waves(TB, RB)
                                   : (SPLIT ? SRE2_P2S_WAVES : SRE2_P2_WAVES))))
void k_pass2(const typename CT<Real>::T* __restrict__ scratch, int NS, int P,
             double* __restrict__ part, const int* __restrict__ scale_exp, const Spec sp,
             int64_t x0) {
    static_assert(!PAIR || (!HERM && !GEN), "row pairs: plain and split M2 forms only");
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
    __shared__ unsigned lh[GEN ? kMaxBins : 1];
    Real lnorm2 = Real(0);
    if constexpr (GEN) {
        hist_clear(lh, sp);
        lnorm2 = hist_lnorm2<Real>(sp);
    }

    const int64_t b = blockIdx.x;
    const int64_t s = b / P;
    const int g = (int)(b % P);
    const int L = NS - HT;  // row bits of pass 1
    const int ntile = 1 << (L - CB);  // column tiles per shift
    const int per = ntile / P;
    const int SH = PAIR ? NS - 1 : NS;  // slab bits of one shift
    const auto rs = buf_rsrc(scratch + ((uint64_t)s << SH), (uint32_t)sizeof(C) << SH);
    // tile element e -> slab offset (e >> CB) * 2^L + (e & CMASK), which adds
    // over disjoint bits: the thread's part once, the register element's part
    // (and the column tile's) as a uniform offset
    const uint32_t base = thread_base<r0.lperm, r0.wave>();
    const uint32_t vb = ((base >> CB) << L) + (base & CMASK);
    // row pairs: the shift's row and column parts, the left-out row bit j,
    // the thread's stored-row (vb0) and partner-row (vb1) address parts and
    // the sign (-1)^popcount(z & xl) of its column bits
    constexpr uint32_t RROW = r0.reg >> CB;
    // the thread-row variant is left out of the plain half-LDS tiles (their
    // registers are full); their row pairs start where x >> L has a register
    // row bit, which for their plans (the top row bits in registers) is
    // x >= 2^(L + lowest register row bit), pair_first_shift
    constexpr bool THR = !half_lds<Real>(TB) || SPLIT;
    static_assert(!PAIR || THR || RROW + (RROW & (0u - RROW)) == (1u << HT),
                  "half-LDS row pairs need the top row bits in registers");
    uint32_t xh = 0, xl = 0, vb0 = 0, vb1 = 0, sT = 0, fm = 0;
    int j = 0;
    if constexpr (PAIR) {
        const uint64_t x = (uint64_t)(x0 + s);
        xh = (uint32_t)(x >> L);
        xl = (uint32_t)x & ((1u << L) - 1u);
        j = half_row_bit(xh, RROW);
        const uint32_t rowT = base >> CB, colT = base & CMASK;
        if constexpr (THR) {
            vb0 = (remove_bit(rowT, j) << L) + colT;
            vb1 = (remove_bit(rowT ^ (xh & ~RROW), j) << L) + colT;
            sT = __builtin_popcount(colT & xl) & 1u;
            fm = 0u - ((rowT >> j) & 1u);
        }
    }
    double acc = 0.0;
    // column transform of one tile and its terms, tiles in ascending order
    auto consume = [&](C (&v)[1 << RB]) {
        run_transform<Real, TB, RB, PK>(lds, v);
        if constexpr (GEN) {
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) acc += gen_terms<Real, HERM>(v[i], sp, lnorm2, lh);
        } else {
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) acc += HERM ? abs4h(v[i]) : abs4(v[i]);
        }
    };
    const int c0 = g * per, c1 = (g + 1) * per;
    // Plain, Hermitian and row-pair tiles that fit the LDS whole load the
    // next tile while transforming this one (two register sets; these
    // kernels are held to two waves per SIMD by their LDS tiles, which leaves
    // the registers; the full-slab split kernel and split tiles above 2^12
    // values have none to spare);
    // barriers wait on LDS only, so the loads stay in flight across the
    // transform.  load_tile(v, ct) fills v with column tile ct.
    constexpr bool PREFETCH = !half_lds<Real>(TB) && (!SPLIT || (PAIR && TB <= 12)) && !GEN;
    auto tiles = [&](auto&& load_tile) {
        if constexpr (PREFETCH) {
            C va[1 << RB], vn[1 << RB];
            load_tile(va, c0);
            for (int ct = c0; ct < c1; ct += 2) {
                if (ct + 1 < c1) load_tile(vn, ct + 1);
                consume(va);
                if (ct + 1 < c1) {
                    if (ct + 2 < c1) load_tile(va, ct + 2);
                    consume(vn);
                }
            }
        } else {
            for (int ct = c0; ct < c1; ++ct) {
                C v[1 << RB];
                load_tile(v, ct);
                consume(v);
            }
        }
    };
    if constexpr (PAIR) {
        if ((RROW >> j) & 1u) {
            with_reg_row_bit<RROW>(j, [&](auto J) {
                tiles([&](C (&v)[1 << RB], int ct) {
                    constexpr int JJ = decltype(J)::value;
                    const uint32_t cto = (uint32_t)ct << CB;
                    uint32_t v0 = vb0, v1 = vb1, st = sT;
                    if constexpr (!THR) {
                        // large tiles: the thread's parts formed per tile from
                        // its id (the empty asm statements keep them there),
                        // so that no register holds them across the
                        // transform; remove_bit is linear over XOR, so the
                        // partner part is the stored part XOR a uniform term
                        uint32_t tb = thread_base<r0.lperm, r0.wave>();
                        uint32_t xt = remove_bit(xh & ~RROW, JJ) << L;
                        asm volatile("" : "+v"(tb), "+s"(xt));
                        v0 = (remove_bit(tb >> CB, JJ) << L) + (tb & CMASK);
                        v1 = v0 ^ xt;
                        st = __builtin_popcount(tb & CMASK & xl) & 1u;
                    }
                    const uint32_t mT = ((st ^ __builtin_popcount(cto & xl)) & 1u) ? kSign : 0u;
                    pair_load_reg<C, RB, r0.reg, CB, JJ>(v, rs, L, v0, v1, xh, xl, cto, mT);
                });
            });
        } else if constexpr (THR) {
            const uint32_t vbt = fm ? vb1 : vb0;
            tiles([&](C (&v)[1 << RB], int ct) {
                const uint32_t cto = (uint32_t)ct << CB;
                const uint32_t mT = ((sT ^ __builtin_popcount(cto & xl)) & 1u) ? kSign : 0u;
                pair_load_thr<C, RB, r0.reg, CB>(j, v, rs, L, vbt, fm, xl, cto, mT);
            });
        } else {
            // half-LDS tiles take row pairs only for shifts whose row part
            // has a register row bit (pair_first_shift); a launch outside
            // that range reports NaN rather than a wrong sum
            acc = __builtin_nan("");
        }
    } else {
        tiles([&](C (&v)[1 << RB], int ct) {
            const uint32_t cto = (uint32_t)ct << CB;
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) {
                const uint32_t r = pdep((uint32_t)i, r0.reg);
                v[i] = load_at<C, NT ? 2 : 0>(rs, vb, cto + ((r >> CB) << L) + (r & CMASK));
            }
        });
    }
    if constexpr (!GEN) {
        if constexpr (HERM) acc *= 16.0;
        if constexpr (SPLIT) acc *= ldexp(1.0, -4 * *scale_exp);
    }
    const double tot = block_sum<T>(acc, red);
    if (threadIdx.x == 0) part[b] = tot;
    if constexpr (GEN) hist_flush(lh, sp);
}

namespace {

template <typename Real, int HT, bool HERM, int SPLIT, bool GEN, bool PAIR>
hipError_t launch_pass2_ht(const void* scratch, int NS, int cs, int P, double* part, const int* se,
                           const Spec& sp, int64_t x0, hipStream_t st) {
    using C = typename CT<Real>::T;
    constexpr int TB = pass2_tb<Real>(HT), RB = Tune<Real>::RB2;
    hipLaunchKernelGGL((k_pass2<Real, HT, TB, RB, HERM, SPLIT, GEN, PAIR>),
                       dim3((unsigned)((int64_t)cs * P)), dim3(1 << (TB - RB)), 0, st,
                       (const C*)scratch, NS, P, part, se, sp, x0);
    return hipGetLastError();
}

template <typename Real, bool HERM, int SPLIT, bool GEN, bool PAIR = false, int... Hs>
hipError_t dispatch_pass2(int HT, const void* scratch, int NS, int cs, int P, double* part,
                          const int* se, const Spec& sp, int64_t x0, hipStream_t st,
                          std::integer_sequence<int, Hs...>) {
    hipError_t e = hipErrorInvalidValue;
    ((HT == Hs + 1
          ? (e = launch_pass2_ht<Real, Hs + 1, HERM, SPLIT, GEN, PAIR>(scratch, NS, cs, P, part,
                                                                       se, sp, x0, st),
             0)
          : 0),
     ...);
    return e;
}

template <typename Real, int... Hs>
int64_t pair_first_shift_of(int N, int split, std::integer_sequence<int, Hs...> hs) {
    const int L = row_bits_of<Real>(N), HT = N - L;
    int64_t first = (int64_t)1 << L;
    if (split == 0 && half_lds<Real>(pass2_tb<Real>(HT))) {
        const uint32_t rrow = pair_pref_of<Real>(HT, split, hs);
        first = (int64_t)1 << (L + __builtin_ctz(rrow));
    }
    return first;
}

}  // namespace

// First shift of the row-pair range of an N-qubit evaluation (split form
// `split`): 2^L, or for the plain half-LDS pass-2 tiles 2^(L + r) with r the
// lowest register row bit of the pass-2 plan, so that x >> L has one.
template <typename Real>
int64_t pair_first_shift(int N, int split) {
    if (N <= Tune<Real>::FMAX || N > max_n_of<Real>()) return (int64_t)1 << N;
    constexpr int HMAX = pass2_max_rows<Real>();
    return pair_first_shift_of<Real>(N, split, std::make_integer_sequence<int, HMAX>{});
}
template int64_t pair_first_shift<float>(int, int);
template int64_t pair_first_shift<double>(int, int);

template <typename Real>
hipError_t launch_pass2(const void* scratch, int N, int slab, int split, int64_t x0, int cs,
                        int P, double* part, const int* se, const Spec* sp, hipStream_t st) {
    if (N <= Tune<Real>::FMAX || N > max_n_of<Real>()) return hipErrorInvalidValue;
    if (slab < kSlabFull || slab > kSlabPairs || split < 0 || split > 2 ||
        (split && (slab == kSlabHerm || sizeof(Real) != 4)) || (sp && slab == kSlabPairs))
        return hipErrorInvalidValue;
    int NS, L;
    slab_geometry<Real>(N, slab, &NS, &L);
    if (slab == kSlabPairs && x0 < pair_first_shift<Real>(N, split)) return hipErrorInvalidValue;
    const bool herm = slab == kSlabHerm;
    if (slab == kSlabPairs) NS = N;  // the kernel takes the full slab's bits
    const int HT = NS - L;
    constexpr int HMAX = pass2_max_rows<Real>();
    constexpr auto hs = std::make_integer_sequence<int, HMAX>{};
    if (sp) {
        if (split || sp->kind < kRedPow || sp->kind > kRedHist ||
            (sp->kind == kRedHist && (!sp->hist || !sp->nrm || sp->nbins < 2 ||
                                      sp->nbins > kMaxBins)))
            return hipErrorInvalidValue;
        if (herm)
            return dispatch_pass2<Real, true, 0, true>(HT, scratch, NS, cs, P, part, se, *sp, x0,
                                                       st, hs);
        return dispatch_pass2<Real, false, 0, true>(HT, scratch, NS, cs, P, part, se, *sp, x0,
                                                    st, hs);
    }
    const Spec none{};
    if (herm)
        return dispatch_pass2<Real, true, 0, false>(HT, scratch, NS, cs, P, part, se, none, x0,
                                                    st, hs);
    if (slab == kSlabPairs) {
        if constexpr (sizeof(Real) == 4) {
            if (split == 1)
                return dispatch_pass2<Real, false, 1, false, true>(HT, scratch, NS, cs, P, part,
                                                                   se, none, x0, st, hs);
            if (split == 2)
                return dispatch_pass2<Real, false, 2, false, true>(HT, scratch, NS, cs, P, part,
                                                                   se, none, x0, st, hs);
        }
        return dispatch_pass2<Real, false, 0, false, true>(HT, scratch, NS, cs, P, part, se, none,
                                                           x0, st, hs);
    }
    if constexpr (sizeof(Real) == 4) {
        if (split == 1)
            return dispatch_pass2<Real, false, 1, false>(HT, scratch, NS, cs, P, part, se, none,
                                                         x0, st, hs);
        if (split == 2)
            return dispatch_pass2<Real, false, 2, false>(HT, scratch, NS, cs, P, part, se, none,
                                                         x0, st, hs);
    }
    return dispatch_pass2<Real, false, 0, false>(HT, scratch, NS, cs, P, part, se, none, x0, st,
                                                 hs);
}

template hipError_t launch_pass2<float>(const void*, int, int, int, int64_t, int, int, double*,
                                        const int*, const Spec*, hipStream_t);
template hipError_t launch_pass2<double>(const void*, int, int, int, int64_t, int, int, double*,
                                         const int*, const Spec*, hipStream_t);

}  // namespace sre2
