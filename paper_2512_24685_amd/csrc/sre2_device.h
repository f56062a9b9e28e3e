// sre2_device.h - device helpers shared by the kernel translation units of
// libsre2: the complex product, the terms of the Pauli sums, slab and buffer
// accesses, register butterflies, LDS transposes and block sums.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sre2_half_map.h"
#include "sre2_plan.h"
#include "sre2_internal.h"

namespace sre2 {

template <typename Real> struct CT;
template <> struct CT<float> { using T = float2; };
template <> struct CT<double> { using T = double2; };

// conj(a) * b.  The imaginary part rounds both products before the
// difference (no fused multiply-add), so that cmul_conj_a(b, a) is exactly
// conj(cmul_conj_a(a, b)): f_x(k ^ x) = conj f_x(k) then holds bit for bit,
// which makes the half slabs of the two-pass path agree with full slabs bit
// for bit.  The real part may
// fuse one product: a.x b.x + a.y b.y with either product fused is the same
// for (a, b) and (b, a), as the same expression fuses the same position
// (the GPU tests compare row-pair and full-slab results bit for bit).
template <typename C>
__device__ __forceinline__ C cmul_conj_a(C a, C b) {
    C r;
    r.x = a.x * b.x + a.y * b.y;
    {
#pragma clang fp contract(off)
        r.y = a.x * b.y - a.y * b.x;
    }
    return r;
}

template <typename C>
__device__ __forceinline__ double abs4(C w) {  // |w|^4 with the square in FP64
    const auto m = w.x * w.x + w.y * w.y;
    const double md = (double)m;
    return md * md;
}

// Hermitian-pair form: 16 (Re^4 + Im^4) of one half-space transform value
// equals the sum of |W|^4 over the two Pauli strings it stands for.  The fused
// square is named, so that every kernel rounds the sum alike.
template <typename C>
__device__ __forceinline__ double abs4h(C w) {
    const double a = (double)(w.x * w.x), b = (double)(w.y * w.y);
    return __builtin_fma(a, a, b * b);
}

constexpr int kHistCopies = 16;  // LDS counters per histogram bin

// Histogram bin of one w = |W|^2: lnorm2 = log2(n^2).
template <typename Real>
__device__ __forceinline__ int hist_bin(Real w, const Spec& sp, Real lnorm2) {
    int b = sp.nbins - 1;
    if (w > Real(0)) {  // NaN-safe: every comparison with NaN selects bin 0
        const Real f = floor(lnorm2 - log2(w) + Real(0.5));
        b = !(f >= Real(0)) ? 0 : (f >= Real(sp.nbins - 1) ? sp.nbins - 1 : (int)f);
    }
    return b;
}

// General reduction (Spec kinds) of NE transformed values: the sum of their
// terms in FP64, or (histogram; HIST) a count in the block's LDS bins and 0.
//  GEN_PLAIN  w = |W|^2 of one Pauli string per value
//  GEN_HERM   the parts stand for two strings with |W| = 2 |Re| and 2 |Im|
// Terms are free of branches (w that are not positive are selected away), one
// loop per kind.  alpha = 3 and 4 are products in FP64 of w: two or three
// operations instead of about 30 (FP32; FP64: far more) for
// exp2(alpha log2 w), and more accurate (N = 15 FP32: 2.0 -> 0.75 ms).
enum GenForm { GEN_PLAIN, GEN_HERM };
template <typename Real, int FORM, bool HIST, int NE, typename C>
__device__ __forceinline__ double gen_sum(const C (&v)[NE], const Spec& sp, Real lnorm2,
                                          unsigned* __restrict__ lh) {
    double acc = 0.0;
    // F: factor of w in the Hermitian form (4, or 1 where the sum takes it)
    const auto over = [&](auto F, auto&& term) {
        constexpr Real f = Real(decltype(F)::value);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            // the empty asm keeps the compiler from forming the squares of all
            // values ahead of the branches below (they would not fit the
            // registers)
            Real x = v[i].x, y = v[i].y;
            asm volatile("" : "+v"(x), "+v"(y));
            if constexpr (FORM == GEN_PLAIN)
                acc += term(x * x + y * y);
            else
                acc += term(f * x * x) + term(f * y * y);
        }
    };
    constexpr std::integral_constant<int, 4> four{};
    constexpr std::integral_constant<int, 1> one{};
    // not positive or NaN: 0
    const auto wide = [](Real w) { return (double)(w > Real(0) ? w : Real(0)); };
    if (HIST && sp.kind == kRedHist) {
        const int copy = threadIdx.x & (kHistCopies - 1);
        over(four, [&](Real w) {
            atomicAdd(&lh[hist_bin<Real>(w, sp, lnorm2) * kHistCopies + copy], 1u);
            return 0.0;
        });
    } else if (sp.kind == kRedShannon) {
        over(four, [](Real w) {
            const Real t = w * log2(w);
            return w > Real(0) ? (double)t : 0.0;
        });
    } else if (sp.ipow == 3) {
        over(one, [&](Real w) {
            const double d = wide(w);
            return d * d * d;
        });
        if constexpr (FORM == GEN_HERM) acc *= 64.0;
    } else if (sp.ipow == 4) {
        over(one, [&](Real w) {
            const double d = wide(w), q = d * d;
            return q * q;
        });
        if constexpr (FORM == GEN_HERM) acc *= 256.0;
    } else {
        const Real alpha = (Real)sp.alpha;
        over(four, [alpha](Real w) {
            const Real t = exp2(alpha * log2(w));
            return w > Real(0) ? (double)t : 0.0;
        });
    }
    return acc;
}

// Block-level histogram bins (GEN kernels with a histogram Spec only): cleared
// at kernel start, added to the global counters at the end.  A state's values
// crowd into a few bins, so that with one counter per bin the lanes of a wave
// queue at the same address (67 M counts at N = 13: about 70 us); each bin has
// kHistCopies counters, neighbouring lanes taking neighbouring ones.
__device__ __forceinline__ void hist_clear(unsigned* lh, const Spec& sp) {
    if (sp.kind == kRedHist) {
        for (int i = threadIdx.x; i < kMaxBins * kHistCopies; i += blockDim.x) lh[i] = 0u;
        __syncthreads();
    }
}
__device__ __forceinline__ void hist_flush(unsigned* lh, const Spec& sp) {
    if (sp.kind == kRedHist) {
        __syncthreads();
        for (int i = threadIdx.x; i < sp.nbins; i += blockDim.x) {
            unsigned n = 0;
            for (int c = 0; c < kHistCopies; ++c) n += lh[i * kHistCopies + c];
            if (n) atomicAdd(&sp.hist[i], (unsigned long long)n);
        }
    }
}
template <typename Real>
__device__ __forceinline__ Real hist_lnorm2(const Spec& sp) {
    return sp.kind == kRedHist ? (Real)(2.0 * log2(*sp.nrm)) : Real(0);
}

// Slab traffic: streamed through the caches (no reuse until the other pass).
#ifndef SRE2_NT_SLAB
#define SRE2_NT_SLAB 1
#endif
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef double f64x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void slab_store(float2* p, float2 v) {
    if constexpr (SRE2_NT_SLAB) {
        f32x2v w = {v.x, v.y};
        __builtin_nontemporal_store(w, reinterpret_cast<f32x2v*>(p));
    } else {
        *p = v;
    }
}
__device__ __forceinline__ void slab_store(double2* p, double2 v) {
    if constexpr (SRE2_NT_SLAB) {
        f64x2v w = {v.x, v.y};
        __builtin_nontemporal_store(w, reinterpret_cast<f64x2v*>(p));
    } else {
        *p = v;
    }
}
// Reads through a buffer resource (base, size in bytes): an address is the
// resource base + a per-thread vector offset + a scalar offset, so a gather
// whose per-element part is uniform across the wave (the register element's
// part of an index) keeps that part in a scalar register and runs no
// per-element address arithmetic on the VALU.  Offsets are 32-bit: psi and
// one shift's slab hold at most 2^26 complex128 values (1 GiB).  AUX is the
// cache policy; 2 marks a streaming (non-temporal) read.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
    // word 3 = 0x00020000: raw (unformatted) 32-bit dword access on gfx9
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                             0x00020000);
}
template <int AUX>
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff,
                                         float2& v) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, AUX);
    __builtin_memcpy(&v, &w, sizeof(v));
}
template <int AUX>
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff,
                                         double2& v) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, AUX);
    __builtin_memcpy(&v, &w, sizeof(v));
}
// Element vidx + sidx of the resource, vidx per thread, sidx uniform.
template <typename C, int AUX = 0>
__device__ __forceinline__ C load_at(__amdgpu_buffer_rsrc_t rs, uint32_t vidx, uint32_t sidx) {
    C v;
    buf_load<AUX>(rs, vidx * (uint32_t)sizeof(C), sidx * (uint32_t)sizeof(C), v);
    return v;
}

// Row bit left out of a half slab (Hermitian pair, row pairs), for the row
// part xh = x >> L (nonzero) of a shift x: the lowest set bit inside `pref`
// when there is one (the rebuilt rows of launch_pass2_images), else the top
// set bit.  Pass 1 then builds only the slab rows with that bit clear.
__device__ __forceinline__ int half_row_bit(uint32_t xh, uint32_t pref) {
    const uint32_t p = xh & pref;
    return p ? __builtin_ctz(p) : 31 - __builtin_clz(xh);
}

// Butterflies over the register bits of `bfly` (a subset of `reg`), one tile
// bit at a time (compile-time recursion keeps every register index constant).
template <int RB, uint32_t REG, uint32_t BFLY, int B = 0, typename C>
__device__ __forceinline__ void butterflies(C (&v)[1 << RB]) {
    if constexpr (B < 32) {
        if constexpr (((BFLY >> B) & 1u) != 0) {
            constexpr int rbit = popc(REG & ((1u << B) - 1u));
#pragma unroll
            for (int i = 0; i < (1 << RB); ++i) {
                if ((i >> rbit) & 1) continue;
                const int j = i | (1 << rbit);
                const C a = v[i], c = v[j];
                v[i].x = a.x + c.x;
                v[i].y = a.y + c.y;
                v[j].x = a.x - c.x;
                v[j].y = a.y - c.y;
            }
        }
        butterflies<RB, REG, BFLY, B + 1>(v);
    }
}

// Tile bits of this thread's elements outside the registers: lane-id bit i
// goes to tile bit (LPERM >> 5i) & 31, the wave id to the bits of WAVE.
template <uint32_t LPERM, uint32_t WAVE>
__device__ __forceinline__ uint32_t thread_base() {
    const uint32_t t = threadIdx.x;
    uint32_t b = pdep(t >> 6, WAVE);
#pragma unroll
    for (int i = 0; i < 6; ++i) b |= ((t >> i) & 1u) << ((LPERM >> (5 * i)) & 31u);
    return b;
}

// LDS slot of register element i, r = pdep(i, REG), for a thread whose own
// slot offset (bytes) is pb_bytes:
//  padded buffer: pad(base | r) = pad(base) + pad(r) (disjoint bits), so
//    pad(r) becomes the instruction's constant offset;
//  swizzled buffer: the bits of swz(r) at or above SB are tile bits of REG,
//    where swz(base) is zero, so swz(base) ^ swz(r) = (swz(base) ^ lo) + hi
//    with lo, hi the parts of swz(r) below and above bit SB: one XOR per
//    distinct lo, and hi is the constant offset.
template <int SB, bool PADDED>
__device__ __forceinline__ uint32_t thread_slot(uint32_t base) {
    return PADDED ? pad16<SB>(base) : swz<SB>(base);
}
template <int SB, bool PADDED, typename C>
__device__ __forceinline__ C* lds_slot(C* lds, uint32_t pb_bytes, uint32_t r) {
    char* b = reinterpret_cast<char*>(lds);
    if constexpr (PADDED) {
        return reinterpret_cast<C*>(b + pb_bytes + pad<SB>(r) * (uint32_t)sizeof(C));
    } else {
        const uint32_t e = swz<SB>(r);
        const uint32_t lo = e & ((1u << SB) - 1u), hi = e & ~((1u << SB) - 1u);
        return reinterpret_cast<C*>(b + hi * (uint32_t)sizeof(C) +
                                    (pb_bytes ^ (lo * (uint32_t)sizeof(C))));
    }
}

// Registers v[OFF + i], i < 2^RB, hold the elements base | pdep(i, REG).
template <int SB, bool PADDED, int RB, uint32_t REG, uint32_t LPERM, uint32_t WAVE, int OFF = 0,
          typename C, int NV>
__device__ __forceinline__ void lds_put(C* lds, const C (&v)[NV]) {
    static_assert(OFF + (1 << RB) <= NV, "registers");
    const uint32_t pb = thread_slot<SB, PADDED>(thread_base<LPERM, WAVE>()) * (uint32_t)sizeof(C);
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i)
        *lds_slot<SB, PADDED>(lds, pb, pdep((uint32_t)i, REG)) = v[OFF + i];
}

template <int SB, bool PADDED, int RB, uint32_t REG, uint32_t LPERM, uint32_t WAVE, int OFF = 0,
          typename C, int NV>
__device__ __forceinline__ void lds_get(const C* lds, C (&v)[NV]) {
    static_assert(OFF + (1 << RB) <= NV, "registers");
    const uint32_t pb = thread_slot<SB, PADDED>(thread_base<LPERM, WAVE>()) * (uint32_t)sizeof(C);
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i)
        v[OFF + i] = *lds_slot<SB, PADDED>(const_cast<C*>(lds), pb, pdep((uint32_t)i, REG));
}

// Sum over the 64 lanes of a wave: DPP exchanges inside each row of 16 lanes
// (XOR partners 1, 2, 7, 15: every lane ends with the row's sum), then the
// four rows in order.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double read_lane(double v, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
    return ((read_lane(v, 0) + read_lane(v, 16)) + read_lane(v, 32)) + read_lane(v, 48);
}

// Sum over a block of NT threads (NT a multiple of 64): a butterfly of
// cross-lane exchanges inside each wave (XOR partners 32, 16, ..., 1, so every
// lane ends with the same wave sum), then the wave sums, added in wave order
// by thread 0 through LDS.  The order is fixed by NT alone.  The result is
// valid in thread 0; `red` needs NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red) {
    static_assert(NT % 64 == 0, "whole waves");
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    constexpr int NW = NT / 64;
    if constexpr (NW == 1) {
        return v;
    } else {
        __syncthreads();  // earlier readers of red are done
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        double t = 0.0;
        if (threadIdx.x == 0)
            for (int w = 0; w < NW; ++w) t += red[w];
        return t;
    }
}

}  // namespace sre2
