// sre2_sim.hip - complex128 state-vector simulator for the quench-dynamics
// workloads (C ABI in include/sre2.h, sre2_sim_*), and the pipeline that
// streams its snapshots into the serving loop.
//
// The simulator owns one device state psi (2^N complex128) and a stream of
// its own.  Operations, all as HIP kernels on that stream:
//   * random product state  prod_i (cos(t_i/2)|0> + e^{i p_i} sin(t_i/2)|1>)
//     (the initial state of the Hamiltonian-quench example);
//   * two-qubit gates       4x4 unitaries on qubit pairs, several per pass, index
//     j = bit(q0) + 2 bit(q1) (the brickwork random-circuit example);
//   * TFIM step             psi <- exp(-i H dt) psi for
//     H = -J sum_{i=0}^{N-2} Z_i Z_{i+1} - hx sum_i X_i - hz sum_i Z_i (open
//     chain), by a Chebyshev expansion of the propagator: with a >= ||H||,
//     exp(-i H dt) = sum_k (2 - [k = 0]) (-i)^k J_k(a dt) T_k(H / a), the T_k
//     from the three-term recurrence T_{k+1} = 2 (H/a) T_k - T_{k-1}; the
//     series is cut where |J_k(a dt)| < 1e-17 beyond k > a dt.
// The pipeline evolves step by step and, after every step, copies the state
// into one of a ring of snapshot buffers and submits it to a server as a
// device input; a ring buffer is reused only once its request is done, so the
// evolution of step t + 1 overlaps the evaluation of the earlier snapshots.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <chrono>
#include <cmath>
#include <new>
#include <thread>
#include <utility>
#include <vector>

#include "../../include/sre2.h"
#include "sre2_internal.h"

using namespace sre2;

namespace {

constexpr int kSimMaxN = 26;
constexpr int kRing = 4;  // snapshot buffers of the pipeline

struct ProductArgs {
    double2 f[2 * kSimMaxN];  // qubit i: cos(theta_i / 2), e^{i phi_i} sin(theta_i / 2)
};

// One pass over the state for several gates: the gates act inside a tile of
// tb qubits (the state's other qubits select the tile), which a workgroup
// holds in LDS.  kTileQubits: 2^11 complex128 = 32 KiB, two workgroups of 512
// threads per CU at N = 20.  kPassGates: the matrices travel in the kernel
// arguments (4 KiB).
#ifndef SRE2_TILE_QUBITS
#define SRE2_TILE_QUBITS 11
#endif
constexpr int kTileQubits = SRE2_TILE_QUBITS;
constexpr int kLowQubits = 3;  // always in the tile: 128 contiguous bytes
constexpr int kPassGates = 14;
struct GatePass {
    int ngates = 0, tb = 0;
    uint32_t mask = 0;              // qubits of the tile
    uint32_t qubit[kSimMaxN] = {};  // tile bits' qubits ascending, then the others
    uint32_t pair[kPassGates] = {}; // tile bits a < b of each gate: a + 256 b
    double2 u[kPassGates][16];      // row-major U[i][j], index bit(a) + 2 bit(b)
};
static_assert(sizeof(GatePass) <= 4000, "kernel arguments");

// Product over the qubits [lo, hi) of the factors that the bits of k select
// (f[2 i] for bit i clear, f[2 i + 1] for set).
__device__ __forceinline__ double2 product_of(const double2* f, uint32_t k, int lo, int hi) {
    double re = 1.0, im = 0.0;
    for (int i = lo; i < hi; ++i) {
        const double2 c = f[2 * i + ((k >> i) & 1)];
        const double r = re * c.x - im * c.y;
        im = re * c.y + im * c.x;
        re = r;
    }
    return make_double2(re, im);
}

// A workgroup writes up to four runs of 256 amplitudes: the product over the low
// eight qubits once per thread, that over the others once per run, one complex
// product per amplitude (N factors per amplitude took 18 us at N = 20; 13 now,
// bound by the 16 MiB it writes).
constexpr int kProductLow = 8, kProductRunBits = 2, kProductRuns = 1 << kProductRunBits;
__global__ __launch_bounds__(1 << kProductLow) void k_product(double2* __restrict__ psi, int N,
                                                              const ProductArgs a) {
    __shared__ double2 f[2 * kSimMaxN], high[kProductRuns];
    const int nl = N < kProductLow ? N : kProductLow;
    const uint32_t first = blockIdx.x * kProductRuns, runs = 1u << (N - nl);
    const uint32_t tid = threadIdx.x;
    // the factors at once: read one by one they cost a memory latency each
    if (tid < 2 * kSimMaxN) f[tid] = a.f[tid];
    __syncthreads();
    if (tid < kProductRuns) high[tid] = product_of(f, (first + tid) << kProductLow, nl, N);
    const double2 low = product_of(f, tid, 0, nl);
    __syncthreads();
    if (tid >= 1u << nl) return;
#pragma unroll
    for (uint32_t r = 0; r < kProductRuns; ++r) {
        if (first + r >= runs) break;
        const double2 h = high[r];
        psi[((first + r) << kProductLow) + tid] =
            make_double2(h.x * low.x - h.y * low.y, h.x * low.y + h.y * low.x);
    }
}

// LDS slot of tile element e: the low four bits XORed with the higher ones, so
// that the four-amplitude groups of any pair of tile bits spread over the banks.
__device__ __forceinline__ uint32_t tile_slot(uint32_t e) {
    return e ^ ((e >> 4) & 15u) ^ ((e >> 8) & 15u);
}

// Row of U times the group's four amplitudes.
__device__ __forceinline__ double2 gate_row(const double2* u, const double2 (&a)[4]) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double2 c = u[j];
        re = __builtin_fma(c.x, a[j].x, re);
        im = __builtin_fma(c.x, a[j].y, im);
        re = __builtin_fma(-c.y, a[j].y, re);
        im = __builtin_fma(c.y, a[j].x, im);
    }
    return make_double2(re, im);
}
// Amplitude of group m with zeros at bits lo < hi.
__device__ __forceinline__ uint32_t group_base(uint32_t m, uint32_t lo, uint32_t hi) {
    m = ((m >> lo) << (lo + 1)) | (m & ((1u << lo) - 1u));
    return ((m >> hi) << (hi + 1)) | (m & ((1u << hi) - 1u));
}

// One gate on the qubits lo < hi, one thread per group of four amplitudes.  A
// pass of one gate takes it in place of k_gates: it has no tile to pass through
// LDS and 260 bytes of arguments instead of 4 KB, which cost the host 0.3 us
// (N <= 20: 7.9 against 8.2 us a call; N = 21: 8.5 against 9.9, N = 22: 21.2
// against 23.1, N = 24: 76.3 against 78.5).  Not on the pair (0, 1), where a
// thread's four amplitudes are neighbours and a wave's loads four lines apart
// each (N = 21: 14.7 against 10.0, N = 24: 88.7 against 80.2).
struct Gate {
    double2 u[16];
};
__global__ __launch_bounds__(256) void k_gate(double2* __restrict__ psi, int N, uint32_t lo,
                                              uint32_t hi, const Gate g) {
    const uint32_t m = blockIdx.x * 256u + threadIdx.x;
    if (m >= 1u << (N - 2)) return;
    const uint32_t k = group_base(m, lo, hi);
    double2 a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        a[j] = psi[k | (uint32_t)(j & 1) << lo | (uint32_t)(j >> 1) << hi];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        psi[k | (uint32_t)(i & 1) << lo | (uint32_t)(i >> 1) << hi] = gate_row(g.u + 4 * i, a);
}

// Applies the gates of one pass in order, each thread one group of four
// amplitudes per gate, through LDS.  What bounds it is the pass over memory
// (N = 20: 16 MiB read and written) and, per gate, 62 FP64 operations and 128
// bytes of LDS traffic per group.  Four waves per SIMD hide the LDS and
// argument loads; the loop body is small on purpose: a variant that held 16
// amplitudes in registers and unrolled each pair of register bits took
// 1.7 us per gate (its code ran once or twice per launch, from a cold
// instruction cache) against 1.1 us.  (One kernel per gate: 7.2 us each.)
__global__ __launch_bounds__(1 << (kTileQubits - 2)) void k_gates(double2* __restrict__ psi, int N,
                                                                  const GatePass ps) {
    constexpr int TBITS = kTileQubits - 2;
    constexpr uint32_t T = 1u << TBITS;
    __shared__ double2 t[1 << kTileQubits];
    const uint32_t tid = threadIdx.x;
    const uint32_t size = 1u << ps.tb;
    uint32_t at = 0;
    for (int b = 0; b < N - ps.tb; ++b) at |= ((blockIdx.x >> b) & 1u) << ps.qubit[ps.tb + b];
#pragma unroll
    for (int b = 0; b < TBITS; ++b)
        if (b < ps.tb) at |= ((tid >> b) & 1u) << ps.qubit[b];
    // the tile bits above the thread's
    const uint32_t u0 = TBITS < ps.tb ? 1u << ps.qubit[TBITS] : 0u;
    const uint32_t u1 = TBITS + 1 < ps.tb ? 1u << ps.qubit[TBITS + 1] : 0u;
    double2 a[4];
    // all loads in flight before the first LDS write; elements above a smaller
    // tile repeat its own addresses and land in slots that nothing stores
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = psi[at | (i & 1 ? u0 : 0u) | (i & 2 ? u1 : 0u)];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[tile_slot(i * T + tid)] = a[i];
    for (int g = 0; g < ps.ngates; ++g) {
        const uint32_t lo = ps.pair[g] & 255u, hi = ps.pair[g] >> 8;
        // insert zero bits at lo, then hi (the threads above a smaller tile
        // work on slots of their own); slots of disjoint bits combine by XOR
        const uint32_t m = group_base(tid, lo, hi);
        const uint32_t s0 = tile_slot(m), sl = tile_slot(1u << lo), sh = tile_slot(1u << hi);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = t[s0 ^ (j & 1 ? sl : 0u) ^ (j & 2 ? sh : 0u)];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            t[s0 ^ (i & 1 ? sl : 0u) ^ (i & 2 ? sh : 0u)] = gate_row(&ps.u[g][4 * i], a);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i * T + tid < size)
            psi[at | (i & 1 ? u0 : 0u) | (i & 2 ? u1 : 0u)] = t[tile_slot(i * T + tid)];
}

// H of the TFIM chain, scaled by 1/a: its diagonal part at basis state k
// (Ising and longitudinal-field energies, Z|0> = |0>); the field along x adds
// -hx times the N single-bit flips.
struct Tfim {
    double J, hx, hz, inv_a;
};
__device__ __forceinline__ double tfim_diag(const Tfim& h, int N, uint32_t k) {
    const int bonds_flipped = (int)__popc((k ^ (k >> 1)) & ((1u << (N - 1)) - 1u));
    const int ones = (int)__popc(k & ((1u << N) - 1u));
    return -h.J * (double)((N - 1) - 2 * bonds_flipped) - h.hz * (double)(N - 2 * ones);
}
// T_{k+1} from h = H T_k and T_{k-1} (first: T_1 = h T_0).
__device__ __forceinline__ double2 cheb_next(double2 h, double2 older, bool first) {
    return first ? h : make_double2(2.0 * h.x - older.x, 2.0 * h.y - older.y);
}
// s + m (-i)^k t, m carrying the sign of the time step.
__device__ __forceinline__ double2 cheb_add(double2 s, double m, int k, double2 t) {
    const double g = k & 2 ? -m : m;
    if (k & 1)
        return make_double2(s.x + g * t.y, s.y - g * t.x);
    return make_double2(s.x + g * t.x, s.y + g * t.y);
}

// One Chebyshev term, N = 8 + AB + NH: writes T_k over T_{k-2} and adds its
// share m (-i)^k T_k to acc (first: k = 1, acc starts as m0 T_0).  A workgroup
// holds 2^AB runs of 256 amplitudes: the flips of the low eight bits come from
// LDS, those of the next AB bits from the thread's own registers, the NH high
// ones from memory, all loads in flight at once (N = 16: one after the other
// they took 4.8 us per term).
template <int NH, int AB>
__global__ __launch_bounds__(256) void k_cheb(const double2* __restrict__ cur,
                                              double2* __restrict__ older,
                                              double2* __restrict__ acc, const Tfim h, double m0,
                                              double m, int k) {
    constexpr int LB = 8 + AB, N = LB + NH, A = 1 << AB;
    __shared__ double2 run[A][256];
    const uint32_t t = threadIdx.x, base = (blockIdx.x << LB) + t;
    const bool first = k == 1;
    double2 c[A], f[A], o[A], s[A];
#pragma unroll
    for (int i = 0; i < A; ++i) c[i] = cur[base + 256 * i];
    double2 far[A][NH];
#pragma unroll
    for (int i = 0; i < A; ++i) {
#pragma unroll
        for (int b = 0; b < NH; ++b) far[i][b] = cur[(base ^ (1u << (LB + b))) + 256 * i];
        o[i] = first ? make_double2(0.0, 0.0) : older[base + 256 * i];
        s[i] = first ? make_double2(0.0, 0.0) : acc[base + 256 * i];
    }
#pragma unroll
    for (int i = 0; i < A; ++i) run[i][t] = c[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < A; ++i) {
        f[i] = make_double2(0.0, 0.0);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const double2 v = run[i][t ^ (1u << b)];
            f[i].x += v.x;
            f[i].y += v.y;
        }
#pragma unroll
        for (int b = 0; b < AB; ++b) {
            f[i].x += c[i ^ (1 << b)].x;
            f[i].y += c[i ^ (1 << b)].y;
        }
#pragma unroll
        for (int b = 0; b < NH; ++b) {
            f[i].x += far[i][b].x;
            f[i].y += far[i][b].y;
        }
        const uint32_t q = base + 256 * i;
        const double d = tfim_diag(h, N, q);
        const double2 hc = make_double2((d * c[i].x - h.hx * f[i].x) * h.inv_a,
                                        (d * c[i].y - h.hx * f[i].y) * h.inv_a);
        const double2 nx = cheb_next(hc, o[i], first);
        older[q] = nx;
        if (first) s[i] = make_double2(m0 * c[i].x, m0 * c[i].y);
        acc[q] = cheb_add(s[i], m, k, nx);
    }
}

// Up to kSmallTerms terms of a state of N <= kSmallMaxN qubits in one launch:
// one workgroup holds T_k, T_{k-1} and the sum in registers and exchanges T_k
// through LDS (two buffers, one barrier per term).  A launch per term is
// bound by the launch (5 us each at N = 10).
constexpr int kSmallMaxN = 11, kSmallTerms = 128;
struct ChebCoef {
    double m[kSmallTerms + 1];
};
__global__ __launch_bounds__(1024) void k_cheb_small(double2* __restrict__ newer,
                                                     double2* __restrict__ older,
                                                     double2* __restrict__ acc, int N,
                                                     const Tfim h, int k0, int count,
                                                     const ChebCoef m) {
    constexpr int A = 1 << (kSmallMaxN - 10);
    __shared__ double2 buf[2][1 << kSmallMaxN];
    const uint32_t size = 1u << N, t = threadIdx.x;
    double2 c[A], o[A], s[A];
    double d[A];
#pragma unroll
    for (int i = 0; i < A; ++i) {
        const uint32_t q = t + 1024 * i;
        c[i] = o[i] = s[i] = make_double2(0.0, 0.0);
        if (q < size) {
            c[i] = newer[q];
            if (k0 > 1) {
                o[i] = older[q];
                s[i] = acc[q];
            } else {
                s[i] = make_double2(m.m[0] * c[i].x, m.m[0] * c[i].y);
            }
        }
        d[i] = tfim_diag(h, N, q);
    }
    for (int j = 0; j < count; ++j) {
        double2* __restrict__ b = buf[j & 1];
#pragma unroll
        for (int i = 0; i < A; ++i) b[t + 1024 * i] = c[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < A; ++i) {
            const uint32_t q = t + 1024 * i;
            double2 f = make_double2(0.0, 0.0);
            for (int g = 0; g < N; ++g) {
                const double2 v = b[q ^ (1u << g)];
                f.x += v.x;
                f.y += v.y;
            }
            const double2 hc = make_double2((d[i] * c[i].x - h.hx * f.x) * h.inv_a,
                                            (d[i] * c[i].y - h.hx * f.y) * h.inv_a);
            const double2 nx = cheb_next(hc, o[i], k0 + j == 1);
            o[i] = c[i];
            c[i] = nx;
            s[i] = cheb_add(s[i], m.m[j + 1], k0 + j, nx);
        }
    }
#pragma unroll
    for (int i = 0; i < A; ++i) {
        const uint32_t q = t + 1024 * i;
        if (q < size) {
            newer[q] = c[i];
            older[q] = o[i];
            acc[q] = s[i];
        }
    }
}

// Bessel functions J_0..J_M(x), x > 0, by Miller's backward recurrence
// J_{k-1} = (2k / x) J_k - J_{k+1} from a start far above x, normalised with
// J_0 + 2 sum_{k>=1} J_{2k} = 1 (Abramowitz & Stegun 9.1.27 and 9.1.46).
std::vector<double> bessel_j(double x, int M) {
    const int start = M + 20 + (int)(10.0 + x);
    std::vector<double> j(start + 2, 0.0);
    j[start + 1] = 0.0;
    j[start] = 1e-300;
    for (int k = start; k >= 1; --k) {
        j[k - 1] = (2.0 * k / x) * j[k] - j[k + 1];
        if (std::fabs(j[k - 1]) > 1e250) {  // rescale to stay in range
            for (int q = k - 1; q <= start; ++q) j[q] *= 1e-250;
        }
    }
    double norm = j[0];
    for (int k = 2; k <= start; k += 2) norm += 2.0 * j[k];
    std::vector<double> out(M + 1);
    for (int k = 0; k <= M; ++k) out[k] = j[k] / norm;
    return out;
}

unsigned product_blocks(int N) {
    const int run_bits = kProductLow + kProductRunBits;
    return N > run_bits ? 1u << (N - run_bits) : 1u;
}
unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

struct sre2_sim {
    int device = 0;
    int N = 0;
    hipStream_t st = nullptr;
    double2* psi = nullptr;
    double2* wb = nullptr;   // Chebyshev T_k
    double2* acc = nullptr;  // Chebyshev sum
    void* ring[kRing] = {};
    size_t ring_bytes = 0;
};

namespace {

struct Guard {
    int prev = -1;
    hipError_t err = hipSuccess;
    explicit Guard(int dev) {
        err = hipGetDevice(&prev);
        if (err == hipSuccess) err = hipSetDevice(dev);
    }
    ~Guard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

int launched() { return hipGetLastError() == hipSuccess ? SRE2_OK : SRE2_EHIP; }

// From N = 18 on a workgroup takes four runs: the flips of ten bits stay on
// chip, at 256 workgroups or more.  From N = 22 on four runs with all their loads in
// flight need more than 256 registers, which leaves one wave per SIMD: two runs
// (N = 22: 116 against 100 us per term, N = 24: 535 against 484).
constexpr int cheb_run_bits(int N) { return N < 18 ? 0 : (N < 22 ? 2 : 1); }
template <int N>
void launch_cheb(sre2_sim* s, const double2* cur, double2* older, const Tfim& h, double m0,
                 double m, int k) {
    constexpr int AB = cheb_run_bits(N);
    hipLaunchKernelGGL((k_cheb<N - 8 - AB, AB>), dim3(1u << (N - 8 - AB)), dim3(256), 0, s->st,
                       cur, older, s->acc, h, m0, m, k);
}
template <int... Ns>
void dispatch_cheb(sre2_sim* s, const double2* cur, double2* older, const Tfim& h, double m0,
                   double m, int k, std::integer_sequence<int, Ns...>) {
    ((s->N == Ns + kSmallMaxN + 1
          ? launch_cheb<Ns + kSmallMaxN + 1>(s, cur, older, h, m0, m, k)
          : void()),
     ...);
}

int tfim_step(sre2_sim* s, double J, double hx, double hz, double dt) {
    const int N = s->N;
    // ||H|| <= |J| (N - 1) + N |(hx, hz)|: a site's field has the norm of the
    // vector (the sum |hx| + |hz| takes 40 terms instead of 35 at N = 16 and
    // the quench example's parameters)
    const double a = std::fabs(J) * (N - 1) + std::hypot(hx, hz) * N;
    if (!(a > 0.0) || dt == 0.0) return SRE2_OK;  // H = 0 or no time: identity
    const double x = a * std::fabs(dt);
    int M = (int)(x + 30.0 + 5.0 * std::cbrt(x));
    const std::vector<double> jb = bessel_j(x, M);
    int K = M;
    while (K > (int)x + 1 && std::fabs(jb[K]) < 1e-17) --K;
    // share of T_k: (2 - [k = 0]) (-i sgn(dt))^k J_k(x) = m_k (-i)^k
    const auto share = [&](int k) {
        return (k == 0 ? 1.0 : 2.0) * (dt < 0 && (k & 1) ? -jb[k] : jb[k]);
    };
    const Tfim h{J, hx, hz, 1.0 / a};
    // psi holds T_0, wb receives T_1; then the newer overwrites the older
    double2 *older = s->wb, *newer = s->psi;
    if (N <= kSmallMaxN) {
        for (int k = 1; k <= K; k += kSmallTerms) {
            const int n = K - k + 1 < kSmallTerms ? K - k + 1 : kSmallTerms;
            ChebCoef m;
            m.m[0] = share(0);
            for (int j = 0; j < n; ++j) m.m[j + 1] = share(k + j);
            hipLaunchKernelGGL(k_cheb_small, dim3(1), dim3(1024), 0, s->st, newer, older, s->acc,
                               N, h, k, n, m);
        }
    } else {
        for (int k = 1; k <= K; ++k) {
            dispatch_cheb(s, newer, older, h, share(0), share(k), k,
                          std::make_integer_sequence<int, kSimMaxN - kSmallMaxN>{});
            double2* t = older;
            older = newer;
            newer = t;
        }
    }
    // the sum is the new state; keep the buffers distinct
    double2* t = s->psi;
    s->psi = s->acc;
    s->acc = t;
    return launched();
}

// Gates in passes of k_gates.  A pass takes, in list order, every gate whose
// qubits fit its tile and that shares no qubit with a gate left for a later
// pass, so gates only move past gates they commute with.  It looks at most
// kLookAhead gates ahead, which bounds the planning per pass.
constexpr int kLookAhead = 256;
int apply_gates(sre2_sim* s, const double* gates, const int* pairs, int count) {
    const int tb = s->N < kTileQubits ? s->N : kTileQubits;
    int todo[kLookAhead];  // the next gates in order; `next` follows them
    int ntodo = 0, next = 0;
    for (;;) {
        while (ntodo < kLookAhead && next < count) todo[ntodo++] = next++;
        if (ntodo == 0) break;
        GatePass ps;
        ps.tb = tb;
        ps.mask = (1u << (s->N < kLowQubits ? s->N : kLowQubits)) - 1u;
        int taken[kPassGates], left = 0;
        uint32_t blocked = 0;
        for (int i = 0; i < ntodo; ++i) {
            const int g = todo[i];
            const uint32_t qs = (1u << pairs[2 * g]) | (1u << pairs[2 * g + 1]);
            if (ps.ngates == kPassGates || (qs & blocked) ||
                __builtin_popcount(ps.mask | qs) > tb) {
                blocked |= qs;
                todo[left++] = g;
            } else {
                ps.mask |= qs;
                taken[ps.ngates++] = g;
            }
        }
        ntodo = left;
        // U with its index bits in the order of the qubits
        const auto matrix = [&](int g, bool swap, double2* u) {
            const double* U = gates + 32 * (size_t)g;
            for (int e = 0; e < 16; ++e) {
                const int r = e >> 2, c = e & 3;
                const int f = swap ? 4 * (r >> 1 | (r & 1) << 1) + (c >> 1 | (c & 1) << 1) : e;
                u[e] = make_double2(U[2 * f], U[2 * f + 1]);
            }
        };
        if (ps.ngates == 1) {
            const int a = pairs[2 * taken[0]], b = pairs[2 * taken[0] + 1];
            const int lo = a < b ? a : b, hi = a < b ? b : a;
            if (hi > 1) {
                Gate g;
                matrix(taken[0], a > b, g.u);
                hipLaunchKernelGGL(k_gate, dim3(blocks_for(int64_t(1) << (s->N - 2))), dim3(256), 0,
                                   s->st, s->psi, s->N, (uint32_t)lo, (uint32_t)hi, g);
                continue;
            }
        }
        for (int q = 0; __builtin_popcount(ps.mask) < tb; ++q) ps.mask |= 1u << q;
        for (int q = 0, b = 0, o = tb; q < s->N; ++q)
            ps.qubit[(ps.mask >> q) & 1u ? b++ : o++] = (uint32_t)q;
        for (int i = 0; i < ps.ngates; ++i) {
            const int* pr = pairs + 2 * taken[i];
            const uint32_t p0 = __builtin_popcount(ps.mask & ((1u << pr[0]) - 1u));
            const uint32_t p1 = __builtin_popcount(ps.mask & ((1u << pr[1]) - 1u));
            const bool swap = p0 > p1;
            ps.pair[i] = swap ? p1 + 256 * p0 : p0 + 256 * p1;
            matrix(taken[i], swap, ps.u[i]);
        }
        hipLaunchKernelGGL(k_gates, dim3(1u << (s->N - tb)), dim3(1 << (kTileQubits - 2)), 0,
                           s->st, s->psi, s->N, ps);
    }
    return launched();
}

int check_pairs(int N, const int* pairs, int count) {
    for (int g = 0; g < count; ++g) {
        const int a = pairs[2 * g], b = pairs[2 * g + 1];
        if (a < 0 || b < 0 || a >= N || b >= N || a == b) return SRE2_EINVAL;
    }
    return SRE2_OK;
}

int copy_state(sre2_sim* s, int dtype, void* dst) {
    const int64_t n = int64_t(1) << s->N;
    if (dtype == SRE2_C128) {
        return hipMemcpyAsync(dst, s->psi, (size_t)n * 16, hipMemcpyDeviceToDevice, s->st) ==
                       hipSuccess
                   ? SRE2_OK
                   : SRE2_EHIP;
    }
    return launch_convert(s->psi, kC128, dst, kC64, n, s->st) == hipSuccess ? SRE2_OK : SRE2_EHIP;
}

// Evolution callback of the pipeline: step t (1-based) of the dynamics.
template <typename Step>
int run_pipeline(sre2_sim* s, sre2_server* srv, int steps, int dtype, double* results, Step step) {
    const size_t bytes = (size_t(1) << s->N) * (dtype == SRE2_C64 ? 8 : 16);
    if (s->ring_bytes < bytes) {
        for (void*& r : s->ring) {
            if (r) (void)hipFree(r);
            r = nullptr;
        }
        s->ring_bytes = 0;
        for (void*& r : s->ring)
            if (hipMalloc(&r, bytes) != hipSuccess) {
                (void)hipGetLastError();
                return SRE2_ENOMEM;
            }
        s->ring_bytes = bytes;
    }
    std::vector<uint64_t> tickets(steps + 1, 0);
    auto wait_done = [&](int t) -> int {
        for (;;) {
            int state = 0;
            double lat = 0.0;
            const int rc = sre2_server_poll(srv, tickets[t], &state, results + SRE2_OUT_LEN * t, &lat);
            if (rc) return rc;
            if (state == SRE2_REQ_DONE) return SRE2_OK;
            if (state == SRE2_REQ_CANCELLED) return SRE2_ECANCELLED;
            if (state == SRE2_REQ_FAILED) return SRE2_EHIP;
            std::this_thread::sleep_for(std::chrono::microseconds(50));
        }
    };
    for (int t = 0; t <= steps; ++t) {
        int rc = SRE2_OK;
        if (t > 0) rc = step(t);
        if (!rc && t >= kRing) rc = wait_done(t - kRing);  // ring slot free again
        void* slot = s->ring[t % kRing];
        if (!rc) rc = copy_state(s, dtype, slot);
        if (!rc && hipStreamSynchronize(s->st) != hipSuccess) rc = SRE2_EHIP;
        if (!rc) rc = sre2_server_submit(srv, slot, s->N, dtype, 1, &tickets[t]);
        if (rc) {
            // let submitted requests finish before the ring may be reused
            for (int q = t - kRing + 1; q < t; ++q)
                if (q >= 0) (void)wait_done(q);
            return rc;
        }
    }
    for (int t = steps - kRing + 1; t <= steps; ++t) {
        if (t < 0) continue;
        const int rc = wait_done(t);
        if (rc) return rc;
    }
    return SRE2_OK;
}

}  // namespace

extern "C" {

int sre2_sim_create(sre2_sim** out, int hip_device, int N) {
    if (!out || hip_device < 0 || N < 2 || N > kSimMaxN) return SRE2_EINVAL;
    Guard g(hip_device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    sre2_sim* s = new (std::nothrow) sre2_sim();
    if (!s) return SRE2_ENOMEM;
    s->device = hip_device;
    s->N = N;
    const size_t bytes = (size_t(1) << N) * sizeof(double2);
    if (hipStreamCreateWithFlags(&s->st, hipStreamNonBlocking) != hipSuccess ||
        hipMalloc((void**)&s->psi, bytes) != hipSuccess ||
        hipMalloc((void**)&s->wb, bytes) != hipSuccess ||
        hipMalloc((void**)&s->acc, bytes) != hipSuccess) {
        (void)hipGetLastError();
        sre2_sim_destroy(s);
        return SRE2_ENOMEM;
    }
    // start in |0...0> (the product state with every theta_i = 0)
    ProductArgs a{};
    for (int i = 0; i < N; ++i) a.f[2 * i] = make_double2(1.0, 0.0);
    hipLaunchKernelGGL(k_product, dim3(product_blocks(N)), dim3(1 << kProductLow), 0, s->st,
                       s->psi, N, a);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s->st) != hipSuccess) {
        sre2_sim_destroy(s);
        return SRE2_EHIP;
    }
    *out = s;
    return SRE2_OK;
}

int sre2_sim_destroy(sre2_sim* s) {
    if (!s) return SRE2_OK;
    Guard g(s->device);
    int rc = g.err == hipSuccess ? SRE2_OK : SRE2_EHIP;
    if (s->st) (void)hipStreamSynchronize(s->st);
    void* bufs[] = {s->psi, s->wb, s->acc, s->ring[0], s->ring[1], s->ring[2], s->ring[3]};
    for (void* b : bufs)
        if (b && hipFree(b) != hipSuccess) rc = SRE2_EHIP;
    if (s->st && hipStreamDestroy(s->st) != hipSuccess) rc = SRE2_EHIP;
    delete s;
    return rc;
}

int sre2_sim_product_state(sre2_sim* s, const double* theta, const double* phi) {
    if (!s || !theta || !phi) return SRE2_EINVAL;
    for (int i = 0; i < s->N; ++i)
        if (!std::isfinite(theta[i]) || !std::isfinite(phi[i])) return SRE2_EINVAL;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    ProductArgs a{};
    for (int i = 0; i < s->N; ++i) {
        const double c = std::cos(0.5 * theta[i]), sn = std::sin(0.5 * theta[i]);
        a.f[2 * i] = make_double2(c, 0.0);
        a.f[2 * i + 1] = make_double2(std::cos(phi[i]) * sn, std::sin(phi[i]) * sn);
    }
    hipLaunchKernelGGL(k_product, dim3(product_blocks(s->N)), dim3(1 << kProductLow), 0, s->st,
                       s->psi, s->N, a);
    return launched();
}

int sre2_sim_apply_gates(sre2_sim* s, const double* gates, const int* pairs, int count) {
    if (!s || count < 0 || (count > 0 && (!gates || !pairs))) return SRE2_EINVAL;
    int rc = check_pairs(s->N, pairs, count);
    if (rc) return rc;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    return apply_gates(s, gates, pairs, count);
}

int sre2_sim_tfim_step(sre2_sim* s, double J, double hx, double hz, double dt) {
    if (!s || !std::isfinite(J) || !std::isfinite(hx) || !std::isfinite(hz) || !std::isfinite(dt))
        return SRE2_EINVAL;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    return tfim_step(s, J, hx, hz, dt);
}

int sre2_sim_state(sre2_sim* s, int dtype, void* dst) {
    if (!s || !dst || (dtype != SRE2_C64 && dtype != SRE2_C128)) return SRE2_EINVAL;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    int rc = copy_state(s, dtype, dst);
    if (!rc && hipStreamSynchronize(s->st) != hipSuccess) rc = SRE2_EHIP;
    return rc;
}

int sre2_sim_run_tfim(sre2_sim* s, sre2_server* srv, double J, double hx, double hz, double dt,
                      int steps, int dtype, double* results) {
    if (!s || !srv || !results || steps < 0 || (dtype != SRE2_C64 && dtype != SRE2_C128) ||
        !std::isfinite(J) || !std::isfinite(hx) || !std::isfinite(hz) || !std::isfinite(dt))
        return SRE2_EINVAL;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    return run_pipeline(s, srv, steps, dtype, results,
                        [&](int) { return tfim_step(s, J, hx, hz, dt); });
}

int sre2_sim_run_circuit(sre2_sim* s, sre2_server* srv, const double* gates, const int* pairs,
                         int gates_per_step, int steps, int dtype, double* results) {
    if (!s || !srv || !results || steps < 0 || gates_per_step < 0 ||
        (steps > 0 && gates_per_step > 0 && (!gates || !pairs)) ||
        (dtype != SRE2_C64 && dtype != SRE2_C128))
        return SRE2_EINVAL;
    int rc = check_pairs(s->N, pairs, gates_per_step);
    if (rc) return rc;
    Guard g(s->device);
    if (g.err != hipSuccess) return SRE2_EHIP;
    return run_pipeline(s, srv, steps, dtype, results, [&](int t) {
        return apply_gates(s, gates + (size_t)32 * gates_per_step * (t - 1), pairs,
                           gates_per_step);
    });
}

}  // extern "C"
