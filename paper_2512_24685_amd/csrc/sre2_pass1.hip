// sre2_pass1.hip - pass 1 of the two-pass transforms (rows, slab write).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_twopass.h"

namespace sre2 {

// ---------------------------------------------------------------------------
// Two-pass, pass 1: row transform over k_lo (TB = L bits) of f_x for a chunk
// of shifts; the slab of one shift holds 2^NS values.  NS = N, or with HERM
// a half slab of NS = N - 1: only the rows whose bit j = half_row_bit(x >> L),
// the top set bit, is clear (x >= 2^L, so that j is a row bit), for the
// Hermitian pair and for the row pairs of the plain and split forms (L that
// of the full slab); pref: see half_row_bit.  Grid (cs, rows): block (s, r)
// takes shift slot s of slab row r; blocks are dispatched with x fastest, so
// neighbouring blocks read the same psi rows.
// ---------------------------------------------------------------------------
template <typename Real, int TB, int RB, bool HERM, int SPLIT>
__global__ __launch_bounds__(1 << (TB - RB))
__attribute__((amdgpu_waves_per_eu(half_lds<Real>(TB) ? half_waves(TB, RB)
                                   : (SPLIT && TB <= 12 ? SRE2_P1S_WAVES : SRE2_P1_WAVES))))
void k_pass1(const typename CT<Real>::T* __restrict__ psi, int NS, int64_t x0, int cs,
             typename CT<Real>::T* __restrict__ scratch, const int* __restrict__ scale_exp,
             uint32_t pref) {
    using C = typename CT<Real>::T;
    constexpr int PK = 2000 + 10000 * SPLIT;
    constexpr Plan P = plan_of<Real, TB, RB, PK>();
    constexpr Round r0 = P.r[0];
    constexpr Round rl = P.r[P.nrounds - 1];
    __shared__ C lds[lds_values(P)];

    (void)cs;
    const uint32_t srow = blockIdx.y;  // row within the slab
    const int64_t s = blockIdx.x;      // shift slot in the chunk
    const uint64_t x = (uint64_t)(x0 + s);
    uint32_t row = srow;
    if constexpr (HERM) row = insert0(srow, half_row_bit((uint32_t)(x >> TB), pref));
    const uint32_t rowbase = row << TB;
    const uint32_t prow = rowbase ^ (uint32_t)(x & ~(uint64_t)((1u << TB) - 1u));  // partner row
    const uint32_t xlo = (uint32_t)(x & ((1u << TB) - 1u));
    const auto rs = buf_rsrc(psi, (uint32_t)sizeof(C) << (NS + (HERM ? 1 : 0)));
    C v[1 << RB];
    {
        // element e = base | r (disjoint bits): psi[rowbase + e] takes the
        // thread part base as vector and rowbase + r as scalar offset, and
        // e ^ xlo = (base ^ (xlo outside REG)) + (r ^ (xlo inside REG)), so
        // the per-element parts are uniform and the per-thread parts are
        // formed once
        const uint32_t base = thread_base<r0.lperm, r0.wave>();
        const uint32_t vb = base ^ (xlo & ~r0.reg), xr = xlo & r0.reg;
#pragma unroll
        for (int i = 0; i < (1 << RB); ++i) {
            const uint32_t r = pdep((uint32_t)i, r0.reg);
            v[i] = cmul_conj_a(load_at<C>(rs, vb, prow + (r ^ xr)), load_at<C>(rs, base, rowbase + r));
        }
        if constexpr (SPLIT) {
            const Real sc = ldexpf(1.0f, *scale_exp);
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) {
                v[i].x *= sc;
                v[i].y *= sc;
            }
        }
    }
    run_transform<Real, TB, RB, PK>(lds, v);
    C* __restrict__ out = scratch + ((uint64_t)s << NS) + ((uint64_t)srow << TB);
    const uint32_t base = thread_base<rl.lperm, rl.wave>();
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) slab_store((out + pdep((uint32_t)i, rl.reg)) + base, v[i]);
}

namespace {

template <typename Real, int TB>
hipError_t launch_pass1_tb(const void* psi, int NS, bool half, int split, int64_t x0, int cs,
                           void* scratch, const int* se, uint32_t pref, hipStream_t st) {
    using C = typename CT<Real>::T;
    constexpr int RB = pass1_rb<Real>(TB, false), RBS = pass1_rb<Real>(TB, true);
    const int64_t rows = (int64_t)1 << (NS - TB);
    if (cs < 1 || rows > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)cs, (unsigned)rows), block(1 << (TB - RB)), blocks(1 << (TB - RBS));
    if (split) {
        if constexpr (sizeof(Real) == 4) {
            if (split == 1 && half)
                hipLaunchKernelGGL((k_pass1<Real, TB, RBS, true, 1>), grid, blocks, 0, st,
                                   (const C*)psi, NS, x0, cs, (C*)scratch, se, pref);
            else if (split == 1)
                hipLaunchKernelGGL((k_pass1<Real, TB, RBS, false, 1>), grid, blocks, 0, st,
                                   (const C*)psi, NS, x0, cs, (C*)scratch, se, pref);
            else if (half)
                hipLaunchKernelGGL((k_pass1<Real, TB, RBS, true, 2>), grid, blocks, 0, st,
                                   (const C*)psi, NS, x0, cs, (C*)scratch, se, pref);
            else
                hipLaunchKernelGGL((k_pass1<Real, TB, RBS, false, 2>), grid, blocks, 0, st,
                                   (const C*)psi, NS, x0, cs, (C*)scratch, se, pref);
        }
    } else if (half)
        hipLaunchKernelGGL((k_pass1<Real, TB, RB, true, 0>), grid, block, 0, st, (const C*)psi,
                           NS, x0, cs, (C*)scratch, se, pref);
    else
        hipLaunchKernelGGL((k_pass1<Real, TB, RB, false, 0>), grid, block, 0, st,
                           (const C*)psi, NS, x0, cs, (C*)scratch, se, pref);
    return hipGetLastError();
}

template <typename Real, int... Ls>
hipError_t dispatch_pass1(int L, const void* psi, int NS, bool half, int split, int64_t x0,
                          int cs, void* scratch, const int* se, uint32_t pref, hipStream_t st,
                          std::integer_sequence<int, Ls...>) {
    hipError_t e = hipErrorInvalidValue;
    ((L == Tune<Real>::ROW + Ls
          ? (e = launch_pass1_tb<Real, Tune<Real>::ROW + Ls>(psi, NS, half, split, x0, cs,
                                                             scratch, se, pref, st),
             0)
          : 0),
     ...);
    return e;
}

}  // namespace

template <typename Real>
hipError_t launch_pass1(const void* psi, int N, int slab, int split, int64_t x0, int cs,
                        void* scratch, const int* se, hipStream_t st) {
    if (N <= Tune<Real>::FMAX || N > max_n_of<Real>()) return hipErrorInvalidValue;
    if (slab < kSlabFull || slab > kSlabImages || split < 0 || split > 2 ||
        (split && (slab == kSlabHerm || sizeof(Real) != 4)))
        return hipErrorInvalidValue;
    int NS, L;
    slab_geometry<Real>(N, slab, &NS, &L);
    const bool half = slab == kSlabHerm || slab == kSlabPairs || slab == kSlabImages;
    const uint32_t pref = slab == kSlabImages ? images_rows(N) : 0u;
    if (half && x0 < ((int64_t)1 << L)) return hipErrorInvalidValue;
    return dispatch_pass1<Real>(
        L, psi, NS, half, split, x0, cs, scratch, se, pref, st,
        std::make_integer_sequence<int, Prec<Real>::MAXTB - Tune<Real>::ROW + 1>{});
}

template hipError_t launch_pass1<float>(const void*, int, int, int, int64_t, int, void*,
                                        const int*, hipStream_t);
template hipError_t launch_pass1<double>(const void*, int, int, int, int64_t, int, void*,
                                         const int*, hipStream_t);

}  // namespace sre2
