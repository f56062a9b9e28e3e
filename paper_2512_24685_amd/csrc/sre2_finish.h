// sre2_finish.h - the end of an evaluation: the sum of S_x, the norm of the
// state, M and the status.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sre2_device.h"
#include "sre2_internal.h"

namespace sre2 {

// out = {M, S, n, status} from the sums: status 0 ok, 1 bad input.
__device__ __forceinline__ void final_out(double S, double n, double bad, int N, int kind,
                                          double alpha, double* __restrict__ out) {
    const bool ok = bad == 0.0 && n > 0.0 && isfinite(n) && isfinite(S);
    const double n2 = n * n;
    double m = NAN;
    if (kind == kRedQuartic)
        m = -log2(S / (ldexp(1.0, N) * n2 * n2));
    else if (kind == kRedPow)  // Eq. 1: log2(S / (2^N n^(2 alpha))) / (1 - alpha)
        m = (log2(S) - (double)N - alpha * log2(n2)) / (1.0 - alpha);
    else if (kind == kRedShannon)  // alpha -> 1, with sum_P w = 2^N n^2
        m = log2(n2) - S / (ldexp(1.0, N) * n2);
    out[0] = ok ? m : NAN;
    out[1] = S;
    out[2] = n;
    out[3] = ok ? 0.0 : 1.0;
}

// The whole end of an evaluation of N <= kFinishMaxN qubits in one workgroup
// (grid y: state of a pack): sum of S_x, FP64 norm and non-finite count of psi,
// M and status.  Small calls are launches and little else: the norm, its
// partials' sum, the sum of S_x and the logarithm as kernels of their own cost
// 2.5 to 4 us each with the gaps between them, this one 2.9 (N = 10) to 6.2
// (N = 14; N = 10 call 21.7 -> 13.4 us).  Beyond N = 14 one workgroup takes
// longer to read the state than the three launches it saves.  Fixed order.
constexpr int kFinishMaxN = 14;
constexpr int kFinishThreads = 1024;
// IT values per thread: 2^N = 1024 IT, or less with IT = 1
template <typename C, int IT, typename PackT>
__global__ __launch_bounds__(kFinishThreads) void k_finish(const C* __restrict__ psi,
                                                           const double* __restrict__ Sx, int N,
                                                           double* __restrict__ out,
                                                           const PackT pk, int kind, double alpha) {
    constexpr int NW = kFinishThreads / 64;
    __shared__ double red[3][NW];
    if constexpr (is_packed<PackT>) {
        psi = (const C*)pk.psi[blockIdx.y];
        Sx = pk_sx(pk.ws[blockIdx.y], pk.N);
        out = pk.out[blockIdx.y];
    }
    double s = 0.0, q = 0.0, bad = 0.0;
    if (IT > 1 || threadIdx.x < 1u << N) {
        C p[IT];
        double v[IT];  // all loads in flight at once
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            p[i] = psi[threadIdx.x + i * kFinishThreads];
            v[i] = Sx[threadIdx.x + i * kFinishThreads];
        }
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const double re = (double)p[i].x, im = (double)p[i].y;
            if (!isfinite(re) || !isfinite(im)) bad += 1.0;
            q += re * re + im * im;
            s += v[i];
        }
    }
    s = wave_sum(s);
    q = wave_sum(q);
    bad = wave_sum(bad);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wave] = s;
        red[1][wave] = q;
        red[2][wave] = bad;
    }
    __syncthreads();
    if (wave == 0) {
        s = wave_sum(lane < NW ? red[0][lane] : 0.0);
        q = wave_sum(lane < NW ? red[1][lane] : 0.0);
        bad = wave_sum(lane < NW ? red[2][lane] : 0.0);
        if (lane == 0) final_out(s, q, bad, N, kind, alpha, out);
    }
}

template <typename C, typename PackT>
hipError_t launch_finish_of(const void* psi, const double* Sx, int N, double* out, const PackT& pk,
                            int count, int kind, double alpha, hipStream_t st) {
    const dim3 grid(1, (unsigned)count), block(kFinishThreads);
    const C* p = (const C*)psi;
    switch (N <= 10 ? 10 : N) {
        case 10:
            k_finish<C, 1, PackT><<<grid, block, 0, st>>>(p, Sx, N, out, pk, kind, alpha);
            break;
        case 11:
            k_finish<C, 2, PackT><<<grid, block, 0, st>>>(p, Sx, N, out, pk, kind, alpha);
            break;
        case 12:
            k_finish<C, 4, PackT><<<grid, block, 0, st>>>(p, Sx, N, out, pk, kind, alpha);
            break;
        case 13:
            k_finish<C, 8, PackT><<<grid, block, 0, st>>>(p, Sx, N, out, pk, kind, alpha);
            break;
        case 14:
            k_finish<C, 16, PackT><<<grid, block, 0, st>>>(p, Sx, N, out, pk, kind, alpha);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
inline hipError_t launch_finish(const void* psi, int dtype, const double* Sx, int N, double* out,
                                const Pack& pk, int kind, double alpha, hipStream_t st) {
    const bool f32 = dtype == kC64;
    if (pk.count)
        return f32 ? launch_finish_of<float2>(psi, Sx, N, out, pk, pk.count, kind, alpha, st)
                   : launch_finish_of<double2>(psi, Sx, N, out, pk, pk.count, kind, alpha, st);
    return f32 ? launch_finish_of<float2>(psi, Sx, N, out, NoPack{}, 1, kind, alpha, st)
               : launch_finish_of<double2>(psi, Sx, N, out, NoPack{}, 1, kind, alpha, st);
}

}  // namespace sre2
