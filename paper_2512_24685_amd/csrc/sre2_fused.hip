// sre2_fused.hip - whole transforms on chip: k_tiny and k_fused (N below the
// half transforms; the split forms below theirs, the BF16 form and the FP16
// form's shift 0 up to the largest tile), and the launcher of every on-chip
// shift sum.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_tile.h"

namespace sre2 {

// ---------------------------------------------------------------------------
// Tiny N (N < RB): one thread per shift.
// ---------------------------------------------------------------------------
template <typename Real, int N, bool GEN, typename PackT>
__global__ __launch_bounds__(64) void k_tiny(const typename CT<Real>::T* __restrict__ psi,
                                             int64_t x_begin, int64_t x_count,
                                             double* __restrict__ S_out,
                                             const PackT pk, const Spec sp) {
    using C = typename CT<Real>::T;
    constexpr int D = 1 << N;
    __shared__ unsigned lh[GEN ? kMaxBins * kHistCopies : 1];
    if constexpr (GEN) {
        hist_clear(lh, sp);
        const Real lnorm2 = hist_lnorm2<Real>(sp);
        const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;
        if (idx < x_count) {
            const uint32_t x = (uint32_t)(x_begin + idx);
            C v[D];
#pragma unroll
            for (int k = 0; k < D; ++k) v[k] = cmul_conj_a(psi[k ^ x], psi[k]);
            butterflies<N, (1u << N) - 1u, (1u << N) - 1u>(v);
            S_out[idx] = gen_sum<Real, GEN_PLAIN, true>(v, sp, lnorm2, lh);
        }
        hist_flush(lh, sp);
        return;
    }
    if constexpr (is_packed<PackT>) {
        psi = (const C*)pk.psi[blockIdx.y];
        S_out = pk_sx(pk.ws[blockIdx.y], N) + x_begin;
    }
    const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (idx >= x_count) return;
    const uint32_t x = (uint32_t)(x_begin + idx);
    C v[D];
#pragma unroll
    for (int k = 0; k < D; ++k) v[k] = cmul_conj_a(psi[k ^ x], psi[k]);
    butterflies<N, (1u << N) - 1u, (1u << N) - 1u>(v);
    double s = 0.0;
#pragma unroll
    for (int z = 0; z < D; ++z) s += abs4(v[z]);
    S_out[idx] = s;
}

// ---------------------------------------------------------------------------
// Fused: whole transforms of NT bits in a 2^TB tile of SPT = 2^(TB-NT) shifts.
// From N = 10 on only the split forms take it (FP16 up to 12 and for shift 0,
// BF16 up to 14; and the FP32 spectrum up to 11): the half transforms of k_half
// do half the work and hold twice the waves (N = 14 FP32 450 -> 150 us, FP16
// 442 -> 156 us, N = 13 FP64 142 -> 60 us per evaluation).
//  HERM = false: NT = N, the tile element (slot j, k) is f_x(k), x = x0 + j.
//  HERM = true : NT = N - 1 (Hermitian pair, x >= 1): with hb the top set bit
//                of x, element (j, k') is f_x(k) for k = k' with a 0 inserted
//                at bit hb, i.e. only the half-space k_hb = 0.  Because
//                f_x(k ^ x) = conj f_x(k), W_x(z) over the full space is twice
//                Re or twice i Im of this half transform, so
//                S_x = 16 sum_z' (Re^4 + Im^4).
// ---------------------------------------------------------------------------
template <typename Real, int NT, int TB, int RB, bool HERM, int SPLIT, bool GEN, typename PackT>
__global__ __launch_bounds__(1 << (TB - RB))
__attribute__((amdgpu_waves_per_eu(SPLIT ? SRE2_FUSEDS_WAVES : SRE2_FUSED_WAVES)))
void k_fused(const typename CT<Real>::T* __restrict__ psi, int64_t x_begin, int64_t x_count,
             double* __restrict__ S_out, const int* __restrict__ scale_exp,
             const PackT pk, const Spec sp) {
    using C = typename CT<Real>::T;
    constexpr int T = 1 << (TB - RB);
    constexpr int PK = 1000 + NT + 10000 * SPLIT;
    constexpr Plan P = plan_of<Real, TB, RB, PK>();
    constexpr Round r0 = P.r[0];
    constexpr Round rl = P.r[P.nrounds - 1];
    constexpr int SPT = 1 << (TB - NT);
    constexpr uint32_t KMASK = (1u << NT) - 1u;
    static_assert((rl.reg & ~KMASK) == 0, "last round: one shift per thread");
    // the buffer also holds the reduction's 2^(TB - RB) doubles
    constexpr int NRED = (1 << (TB - RB)) * (int)sizeof(double) / (int)sizeof(C);
    constexpr int NL = lds_values(P);
    __shared__ C lds[NL > NRED ? NL : NRED];
    __shared__ unsigned lh[GEN ? kMaxBins * kHistCopies : 1];
    double* red = reinterpret_cast<double*>(lds);
    if constexpr (is_packed<PackT>) {
        psi = (const C*)pk.psi[blockIdx.y];
        S_out = pk_sx(pk.ws[blockIdx.y], pk.N) + x_begin;
        scale_exp = pk_se(pk.ws[blockIdx.y], pk.N);
    }
    Real lnorm2 = Real(0);
    if constexpr (GEN) {
        hist_clear(lh, sp);
        lnorm2 = hist_lnorm2<Real>(sp);
    }

    const int se = SPLIT ? *scale_exp : 0;
    const Real sc = SPLIT ? ldexpf(1.0f, se) : Real(1);
    const double unscale = SPLIT ? ldexp(1.0, -4 * se) : 1.0;
    const int64_t ntiles = (x_count + SPT - 1) / SPT;
    // one shift per tile (the split forms from N = 12 on): k = e = base | r
    // (disjoint bits) does not depend on the tile, so psi[k] is read once per
    // workgroup and kept in registers over the tiles the workgroup takes
    constexpr bool ONE = SPT == 1;
    static_assert(!ONE || (sizeof(Real) == 4 && !HERM), "the half transforms take the others");
    const auto rs = buf_rsrc(psi, (uint32_t)sizeof(C) << (NT + (HERM ? 1 : 0)));
    C psik[ONE ? (1 << RB) : 1];
    if constexpr (ONE) {
        const uint32_t base = thread_base<r0.lperm, r0.wave>();
#pragma unroll
        for (int i = 0; i < (1 << RB); ++i) psik[i] = load_at<C>(rs, base, pdep((uint32_t)i, r0.reg));
    }
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t x0 = x_begin + tile * SPT;  // first shift of the tile
        C v[1 << RB];
        if constexpr (ONE) {
            // as in pass 1, k ^ x = (base ^ (x outside REG)) + (r ^ (x inside
            // REG)), so the per-element address parts are uniform
            const uint32_t x = (uint32_t)x0;
            const uint32_t base = thread_base<r0.lperm, r0.wave>();
            const uint32_t vb = base ^ (x & ~r0.reg), xr = x & r0.reg;
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) {
                const uint32_t r = pdep((uint32_t)i, r0.reg);
                v[i] = cmul_conj_a(load_at<C>(rs, vb, r ^ xr), psik[i]);
                if constexpr (SPLIT) {
                    v[i].x *= sc;
                    v[i].y *= sc;
                }
            }
        } else {
            const uint32_t base = thread_base<r0.lperm, r0.wave>();
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) {
                const uint32_t e = base | pdep((uint32_t)i, r0.reg);
                const int64_t j = e >> NT;  // shift slot in the tile
                if (tile * SPT + j < x_count) {
                    const uint32_t x = (uint32_t)(x0 + j);
                    uint32_t k = e & KMASK;
                    if constexpr (HERM) k = insert0(k, 31u - __clz(x));
                    v[i] = cmul_conj_a(psi[k ^ x], psi[k]);
                    if constexpr (SPLIT) {
                        v[i].x *= sc;
                        v[i].y *= sc;
                    }
                } else {
                    v[i].x = 0;
                    v[i].y = 0;
                }
            }
        }
        run_transform<Real, TB, RB, PK>(lds, v);
        double s = 0.0;
        if constexpr (GEN) {
            // this thread's values belong to one shift slot (the last round's
            // registers lie inside the transform bits); empty slots of the
            // last tile hold zeros that must not enter the histogram
            const int64_t slot = thread_base<rl.lperm, rl.wave>() >> NT;
            if (tile * SPT + slot < x_count)
                s = gen_sum<Real, HERM ? GEN_HERM : GEN_PLAIN, true>(v, sp, lnorm2, lh);
        } else {
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) s += HERM ? abs4h(v[i]) : abs4(v[i]);
            if constexpr (HERM) s *= 16.0;
            if constexpr (SPLIT) s *= unscale;
        }
        // thread order index: tile bits outside the last round's registers,
        // compressed; its top TB-NT bits are the shift slot.
        const uint32_t q = pext(thread_base<rl.lperm, rl.wave>(), ((1u << TB) - 1u) & ~rl.reg);
        __syncthreads();
        red[q] = s;
        seg_tree<T>(red, T / SPT);
        if (threadIdx.x < SPT) {
            const int64_t j = threadIdx.x;
            if (tile * SPT + j < x_count) S_out[tile * SPT + j] = red[j * (T / SPT)];
        }
    }
    if constexpr (GEN) hist_flush(lh, sp);
}

namespace {

// Workgroups of `threads` threads of `kernel` the current device holds at
// once (CUs x occupancy); 32768 if the runtime cannot say.
int64_t resident_workgroups(const void* kernel, int threads) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess ||
        cus < 1 || per < 1)
        return 32768;
    return (int64_t)cus * per;
}

template <typename Real, int N, bool GEN>
hipError_t launch_tiny_n(const void* psi, int64_t x0, int64_t xc, double* S,
                         const Pack& pk, const Spec& sp, hipStream_t st) {
    using C = typename CT<Real>::T;
    const int64_t blocks = (xc + 63) / 64;
    if constexpr (!GEN) {
        if (pk.count) {
            k_tiny<Real, N, GEN, Pack><<<dim3((unsigned)blocks, (unsigned)pk.count), 64, 0, st>>>(
                (const C*)psi, x0, xc, S, pk, sp);
            return hipGetLastError();
        }
    }
    k_tiny<Real, N, GEN, NoPack><<<dim3((unsigned)blocks), 64, 0, st>>>((const C*)psi, x0, xc, S,
                                                                        NoPack{}, sp);
    return hipGetLastError();
}

template <typename Real, int NT, bool HERM, int SPLIT, bool GEN>
hipError_t launch_fused_nt(const void* psi, int64_t x0, int64_t xc, double* S, const int* se,
                           const Pack& pk, const Spec& sp, hipStream_t st) {
    using C = typename CT<Real>::T;
    constexpr int TB = fused_tb<Real>(NT), RB = fused_rb<Real>(NT, SPLIT != 0);
    constexpr int SPT = 1 << (TB - NT);
    const int64_t ntiles = (xc + SPT - 1) / SPT;
    // Tiles of one shift keep psi[k] in registers, which amortises its reads over
    // the tiles a workgroup takes: their grid is twice the workgroups the GPU holds
    // at once (queried once per kernel; whole tiles of N = 14 took 0.58 ms with
    // one tile per workgroup, 0.44 so), the others take one tile per workgroup up
    // to 65536 workgroups.
    int64_t cap = 65536;
    if constexpr (SPT == 1) {
        static const int64_t resident = resident_workgroups(
            reinterpret_cast<const void*>(&k_fused<Real, NT, TB, RB, HERM, SPLIT, GEN, NoPack>),
            1 << (TB - RB));
        cap = 2 * resident;
    }
    const int64_t grid = ntiles < cap ? ntiles : cap;
    const dim3 block(1 << (TB - RB));
    if constexpr (!GEN) {
        if (pk.count) {
            k_fused<Real, NT, TB, RB, HERM, SPLIT, GEN, Pack>
                <<<dim3((unsigned)grid, (unsigned)pk.count), block, 0, st>>>((const C*)psi, x0, xc,
                                                                            S, se, pk, sp);
            return hipGetLastError();
        }
    }
    k_fused<Real, NT, TB, RB, HERM, SPLIT, GEN, NoPack><<<dim3((unsigned)grid), block, 0, st>>>(
        (const C*)psi, x0, xc, S, se, NoPack{}, sp);
    return hipGetLastError();
}

template <typename Real, bool GEN, int... Ns>
hipError_t dispatch_tiny(int N, const void* psi, int64_t x0, int64_t xc, double* S,
                         const Pack& pk, const Spec& sp, hipStream_t st,
                         std::integer_sequence<int, Ns...>) {
    hipError_t e = hipErrorInvalidValue;
    ((N == Ns + 1 ? (e = launch_tiny_n<Real, Ns + 1, GEN>(psi, x0, xc, S, pk, sp, st), 0) : 0),
     ...);
    return e;
}

template <typename Real, bool HERM, int SPLIT, bool GEN, int... Ns>
hipError_t dispatch_fused(int NT, const void* psi, int64_t x0, int64_t xc, double* S,
                          const int* se, const Pack& pk, const Spec& sp, hipStream_t st,
                          std::integer_sequence<int, Ns...>) {
    constexpr int RB = Tune<Real>::RBF;
    hipError_t e = hipErrorInvalidValue;
    ((NT == Ns + RB
          ? (e = launch_fused_nt<Real, Ns + RB, HERM, SPLIT, GEN>(psi, x0, xc, S, se, pk, sp, st),
             0)
          : 0),
     ...);
    return e;
}

}  // namespace

template <typename Real, bool GEN>
hipError_t shift_kernel_gen(const void* psi, int N, bool herm, int split, int64_t x0,
                            int64_t xc, double* S, const int* se, const Pack& pk, const Spec& sp,
                            hipStream_t st) {
    // above FMAX the half transforms take the plain and Hermitian forms
    constexpr int RB = Tune<Real>::RBF;
    constexpr int FMAX = (GEN ? half_hist_min<Real>() : Tune<Real>::HMIN) - 1;
    if (herm) {
        if (x0 < 1 || N - 1 < RB) return hipErrorInvalidValue;
        return dispatch_fused<Real, true, 0, GEN>(N - 1, psi, x0, xc, S, se, pk, sp, st,
                                                      std::make_integer_sequence<int, FMAX - RB>{});
    }
    if (N < RB)
        return dispatch_tiny<Real, GEN>(N, psi, x0, xc, S, pk, sp, st,
                                        std::make_integer_sequence<int, RB - 1>{});
    if constexpr (sizeof(Real) == 4 && !GEN) {
        constexpr auto ns = std::make_integer_sequence<int, Tune<Real>::FMAX - RB + 1>{};
        if (split == 1)
            return dispatch_fused<Real, false, 1, false>(N, psi, x0, xc, S, se, pk, sp, st, ns);
        if (split == 2)
            return dispatch_fused<Real, false, 2, false>(N, psi, x0, xc, S, se, pk, sp, st, ns);
    }
    return dispatch_fused<Real, false, 0, GEN>(N, psi, x0, xc, S, se, pk, sp, st,
                                                   std::make_integer_sequence<int, FMAX - RB + 1>{});
}

template <typename Real>
hipError_t launch_shift_kernel(const void* psi, int N, bool herm, int split, int64_t x0,
                               int64_t xc, double* S, const int* se, const Pack& pk,
                               const Spec* sp, hipStream_t st) {
    const bool hist = sp && sp->kind == kRedHist;
    // (the split forms' shift 0 goes through k_fused)
    const bool half = split  ? split == 1 && x0 > 0 && N >= Tune<Real>::HSPLIT &&
                                  N <= Tune<Real>::HMAX
                      : hist ? N >= half_hist_min<Real>() && N <= half_hist_max<Real>()
                             : N >= Tune<Real>::HMIN && N <= Tune<Real>::HMAX;
    if ((N > Tune<Real>::FMAX && !half) || split < 0 || split > 2 ||
        (split && (herm || sizeof(Real) != 4)) || pk.count > kMaxPack)
        return hipErrorInvalidValue;
    if (sp) {
        if (split || pk.count || sp->kind < kRedPow || sp->kind > kRedHist ||
            (hist && (!sp->hist || !sp->nrm || sp->nbins < 2 || sp->nbins > kMaxBins)))
            return hipErrorInvalidValue;
    }
    if (half) return launch_half<Real>(psi, N, herm, split, x0, xc, S, se, pk, sp, st);
    if (sp)
        return shift_kernel_gen<Real, true>(psi, N, herm, split, x0, xc, S, se, pk, *sp, st);
    return shift_kernel_gen<Real, false>(psi, N, herm, split, x0, xc, S, se, pk, Spec{}, st);
}

template hipError_t launch_shift_kernel<float>(const void*, int, bool, int, int64_t, int64_t,
                                               double*, const int*, const Pack&, const Spec*,
                                               hipStream_t);
template hipError_t launch_shift_kernel<double>(const void*, int, bool, int, int64_t, int64_t,
                                                double*, const int*, const Pack&, const Spec*,
                                                hipStream_t);

}  // namespace sre2
