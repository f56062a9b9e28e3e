// sre2_kernels.hip - gfx950 kernels for the XOR-FWHT evaluation of the
// second-order stabilizer Renyi entropy (arXiv:2512.24685, Algorithm 1 and
// Eq. final1):
//
//   S_x = sum_z |W_x(z)|^4,  W_x = FWHT_k( conj(psi[k ^ x]) * psi[k] ),
//   S   = sum_x S_x,          M2  = -log2( S / (2^N n^4) ),  n = sum_k |psi[k]|^2.
//
// W_x(z) equals <psi| X^x Z^z |psi> (Eq. Pauli_expect), so every W is a Pauli
// expectation.  Shifts x are independent units of work (main text: the shift
// loop is parallel); each kernel below owns a set of shifts or a slice of one.
//
// The shift sums themselves are in their own files:
//  sre2_fused.hip  k_tiny (N < RB: one thread per shift) and k_fused
//                  (RB <= N: 2^(TB-N) complete shifts in a 2^TB tile; N below
//                  the half transforms, the split forms, the spectrum).
//  sre2_half.hip   k_half: a half transform per workgroup, on chip up to
//                  N = 16 (FP32) / 15 (FP64).
//  sre2_pass1.hip  k_pass1: row transform over the low TB bits of k, f_x built
//                  on the fly from psi, written to a scratch slab (for shifts
//                  x >= 2^TB only half its rows: Hermitian pair, row pairs).
//  sre2_pass2.hip  k_pass2: column transform over the high N-TB bits, |W|^4
//                  and a per-workgroup FP64 partial sum; nothing is written
//                  back.  Half slabs are transformed as they are: 2 Re and
//                  2i Im of the result are the values of the shift.
// Here:
//  k_convert / k_norm_part / k_sum_part / k_final: input staging, FP64 norm,
//              fixed-order FP64 reductions and the logarithm (N above the
//              range of k_finish, sre2_finish.h, which does the last three).
//  k_moment_part / k_moment_final: sum |psi|^2, sum |psi|^4 and non-finite
//              count of an input (sre2_moments).
//
// Forms: FP32 or FP64 butterflies; the Hermitian pair (half the transform
// of shifts x >= 1); the split forms, whose H_16 factors run on the matrix
// cores with FP16 or BF16 hi/lo halves (SPLIT = 1, 2).
//
// Accumulation: |W|^2 is formed in the working precision, squared and summed
// in FP64 per element; per-thread sums are combined by fixed-shape trees, so a
// result depends only on (psi, N, form), never on scheduling.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "sre2_internal.h"
#include "sre2_device.h"
#include "sre2_finish.h"

namespace sre2 {

// ---------------------------------------------------------------------------
// Staging and reductions.
// ---------------------------------------------------------------------------
template <typename Src, typename Dst>
__global__ void k_convert(const Src* __restrict__ in, Dst* __restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        Dst d;
        d.x = in[i].x;
        d.y = in[i].y;
        out[i] = d;
    }
}

constexpr int kRedThreads = 256;
static_assert(kRedThreads <= kMaxRed, "reduction blocks");

// part[b] = sum of |psi|^2 over block b's fixed range; flag[b] = non-finite seen.
template <typename C, typename PackT>
__global__ __launch_bounds__(kRedThreads) void k_norm_part(const C* __restrict__ psi, int64_t n,
                                                           int64_t per_block,
                                                           double* __restrict__ part,
                                                           double* __restrict__ flag,
                                                           const PackT pk) {
    __shared__ double red[kRedThreads];
    if constexpr (is_packed<PackT>) {
        psi = (const C*)pk.psi[blockIdx.y];
        part = pk_npart(pk.ws[blockIdx.y], pk.N);
        flag = pk_nflag(pk.ws[blockIdx.y], pk.N);
    }
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < n ? lo + per_block : n;
    double s = 0.0;
    int bad = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kRedThreads) {
        const double re = (double)psi[i].x, im = (double)psi[i].y;
        if (!isfinite(re) || !isfinite(im)) bad = 1;
        s += re * re + im * im;
    }
    const double tot = block_sum<kRedThreads>(s, red);
    const double nbad = block_sum<kRedThreads>(bad ? 1.0 : 0.0, red);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = tot;
        flag[blockIdx.x] = nbad;
    }
}

// Moments of the input as given, per block over the same fixed ranges as
// k_norm_part: m[b] = sum |psi|^2, m[K + b] = sum |psi|^4 (the inverse
// participation ratio's numerator), m[2K + b] = count of non-finite
// amplitudes, K = kMaxRed; all in FP64.
template <typename C>
__global__ __launch_bounds__(kRedThreads) void k_moment_part(const C* __restrict__ psi, int64_t n,
                                                             int64_t per_block,
                                                             double* __restrict__ m) {
    __shared__ double red[kRedThreads];
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < n ? lo + per_block : n;
    double s2 = 0.0, s4 = 0.0, bad = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kRedThreads) {
        const double re = (double)psi[i].x, im = (double)psi[i].y;
        if (!isfinite(re) || !isfinite(im)) bad += 1.0;
        const double q = re * re + im * im;
        s2 += q;
        s4 += q * q;
    }
    const double t2 = block_sum<kRedThreads>(s2, red);
    const double t4 = block_sum<kRedThreads>(s4, red);
    const double tb = block_sum<kRedThreads>(bad, red);
    if (threadIdx.x == 0) {
        m[blockIdx.x] = t2;
        m[kMaxRed + blockIdx.x] = t4;
        m[2 * kMaxRed + blockIdx.x] = tb;
    }
}

// out[j] = sum over b < nb of m[j K + b] in b order, j = 0, 1, 2.
__global__ void k_moment_final(const double* __restrict__ m, int nb, double* __restrict__ out) {
    const int j = threadIdx.x;
    if (j >= 3) return;
    double a = 0.0;
    for (int b = 0; b < nb; ++b) a += m[j * kMaxRed + b];
    out[j] = a;
}

// part[b] = sum of v over block b's fixed range (optionally with stride-P
// grouping: entry x*P+p belongs to shift x; Sx, when non-null, receives
// sum_p v[x*P+p] in p order).
__global__ __launch_bounds__(kRedThreads) void k_sum_part(const double* __restrict__ v,
                                                          int64_t nshift, int P,
                                                          int64_t per_block,
                                                          double* __restrict__ part,
                                                          double* __restrict__ Sx) {
    __shared__ double red[kRedThreads];
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < nshift ? lo + per_block : nshift;
    double s = 0.0;
    for (int64_t x = lo + threadIdx.x; x < hi; x += kRedThreads) {
        double sx = 0.0;
        for (int p = 0; p < P; ++p) sx += v[x * P + p];
        if (Sx) Sx[x] = sx;
        s += sx;
    }
    const double tot = block_sum<kRedThreads>(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Sx[s] = sum_p part[s*P + p] in p order (one thread per shift).
__global__ __launch_bounds__(256) void k_group_sum(const double* __restrict__ part, int64_t ns,
                                                   int P, double* __restrict__ Sx) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= ns) return;
    double a = 0.0;
    for (int p = 0; p < P; ++p) a += part[s * P + p];
    Sx[s] = a;
}

// out[0] = M2, out[1] = S, out[2] = n, out[3] = status (0 ok, 1 bad input).
__global__ __launch_bounds__(kRedThreads) void k_final(const double* __restrict__ spart, int ns,
                                                       const double* __restrict__ npart,
                                                       const double* __restrict__ nflag, int nn,
                                                       int N, double* __restrict__ out, int kind,
                                                       double alpha) {
    __shared__ double red[kRedThreads];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int i = threadIdx.x; i < ns; i += kRedThreads) a += spart[i];
    for (int i = threadIdx.x; i < nn; i += kRedThreads) {
        b += npart[i];
        c += nflag[i];
    }
    const double S = block_sum<kRedThreads>(a, red);
    const double n = block_sum<kRedThreads>(b, red);
    const double bad = block_sum<kRedThreads>(c, red);
    if (threadIdx.x == 0) final_out(S, n, bad, N, kind, alpha, out);
}

// s = 14 - ceil(log2 n) from the norm partials (0 when n is not positive and
// finite): with every |value| of a transform bounded by n, the scaled values
// of the split form stay below 2^14, inside FP16's range.
template <typename PackT>
__global__ void k_split_scale(const double* __restrict__ npart, int nb, int* __restrict__ se,
                              const PackT pk) {
    if (threadIdx.x != 0) return;
    if constexpr (is_packed<PackT>) {
        npart = pk_npart(pk.ws[blockIdx.y], pk.N);
        se = pk_se(pk.ws[blockIdx.y], pk.N);
    }
    double n = 0.0;
    for (int i = 0; i < nb; ++i) n += npart[i];
    int s = 0;
    if (n > 0.0 && isfinite(n)) {
        s = 14 - (int)ceil(log2(n));
        s = s < -100 ? -100 : (s > 100 ? 100 : s);
    }
    *se = s;
}

hipError_t launch_split_scale(const double* npart, int nb, int* se, const Pack& pk, hipStream_t st) {
    if (pk.count)
        k_split_scale<<<dim3(1, (unsigned)pk.count), 64, 0, st>>>(npart, nb, se, pk);
    else
        k_split_scale<<<1, 64, 0, st>>>(npart, nb, se, NoPack{});
    return hipGetLastError();
}

hipError_t launch_convert(const void* in, int in_dtype, void* out, int out_dtype, int64_t n,
                          hipStream_t st) {
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (in_dtype == kC128 && out_dtype == kC64)
        hipLaunchKernelGGL((k_convert<double2, float2>), dim3(blocks), dim3(256), 0, st,
                           (const double2*)in, (float2*)out, n);
    else if (in_dtype == kC64 && out_dtype == kC128)
        hipLaunchKernelGGL((k_convert<float2, double2>), dim3(blocks), dim3(256), 0, st,
                           (const float2*)in, (double2*)out, n);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename C>
hipError_t launch_norm_of(const void* psi, int64_t n, int nblocks, double* part, double* flag,
                          const Pack& pk, hipStream_t st) {
    const int64_t per = (n + nblocks - 1) / nblocks;
    const C* p = (const C*)psi;
    if (pk.count)
        k_norm_part<C><<<dim3(nblocks, pk.count), kRedThreads, 0, st>>>(p, n, per, part, flag, pk);
    else
        k_norm_part<C><<<nblocks, kRedThreads, 0, st>>>(p, n, per, part, flag, NoPack{});
    return hipGetLastError();
}

hipError_t launch_norm(const void* psi, int dtype, int64_t n, int nblocks, double* part,
                       double* flag, const Pack& pk, hipStream_t st) {
    return dtype == kC64 ? launch_norm_of<float2>(psi, n, nblocks, part, flag, pk, st)
                         : launch_norm_of<double2>(psi, n, nblocks, part, flag, pk, st);
}

hipError_t launch_moments(const void* psi, int dtype, int64_t n, int nblocks, double* m,
                          double* out, hipStream_t st) {
    if (nblocks < 1 || nblocks > kMaxRed) return hipErrorInvalidValue;
    const int64_t per = (n + nblocks - 1) / nblocks;
    if (dtype == kC64)
        hipLaunchKernelGGL((k_moment_part<float2>), dim3(nblocks), dim3(kRedThreads), 0, st,
                           (const float2*)psi, n, per, m);
    else
        hipLaunchKernelGGL((k_moment_part<double2>), dim3(nblocks), dim3(kRedThreads), 0, st,
                           (const double2*)psi, n, per, m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_moment_final, dim3(1), dim3(64), 0, st, m, nblocks, out);
    return hipGetLastError();
}

hipError_t launch_sum(const double* v, int64_t nshift, int P, int nblocks, double* part,
                      double* Sx, const Pack& pk, hipStream_t st) {
    if (pk.count) return hipErrorInvalidValue;  // packed sizes: finish (sre2_finish.h)
    const int64_t per = (nshift + nblocks - 1) / nblocks;
    hipLaunchKernelGGL(k_sum_part, dim3(nblocks), dim3(kRedThreads), 0, st, v, nshift, P, per,
                       part, Sx);
    return hipGetLastError();
}

hipError_t launch_group_sum(const double* part, int64_t ns, int P, double* Sx, hipStream_t st) {
    hipLaunchKernelGGL(k_group_sum, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, st, part, ns,
                       P, Sx);
    return hipGetLastError();
}

hipError_t launch_final(const double* spart, int ns, const double* npart, const double* nflag,
                        int nn, int N, double* out, const Pack& pk, int kind, double alpha,
                        hipStream_t st) {
    if (pk.count) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_final, dim3(1), dim3(kRedThreads), 0, st, spart, ns, npart, nflag, nn, N,
                       out, kind, alpha);
    return hipGetLastError();
}

__global__ void k_norm_total(const double* __restrict__ npart, int nb, double* __restrict__ nrm) {
    if (threadIdx.x != 0) return;
    double n = 0.0;
    for (int i = 0; i < nb; ++i) n += npart[i];
    *nrm = n;
}

hipError_t launch_norm_total(const double* npart, int nb, double* nrm, hipStream_t st) {
    hipLaunchKernelGGL(k_norm_total, dim3(1), dim3(64), 0, st, npart, nb, nrm);
    return hipGetLastError();
}

__global__ void k_zero_u64(unsigned long long* __restrict__ p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0ull;
}

hipError_t launch_zero_u64(unsigned long long* p, int count, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_u64, dim3((count + 63) / 64), dim3(64), 0, st, p, count);
    return hipGetLastError();
}

}  // namespace sre2
