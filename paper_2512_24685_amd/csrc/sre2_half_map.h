// sre2_half_map.h - index maps of the on-chip half transforms (k_half): their
// plans, which values of a shift they hold, and the bits of shift 0.
// Host-compilable, so that the maps can be checked without a GPU.
#pragma once
#include "sre2_geometry.h"

namespace sre2 {

// Insert a zero bit at position `hb` of `v`.
__host__ __device__ constexpr uint32_t insert0(uint32_t v, uint32_t hb) {
    return ((v >> hb) << (hb + 1)) | (v & ((1u << hb) - 1u));
}

// Plan of the half transform of NT bits (split form s: H_16 factors on the
// matrix cores, as in the other kernels of the split forms).  SB = 5 for both
// precisions: the buffer holds one real part.
constexpr int kHalfSB = 5;
template <int NT, int RB, int SPLIT>
__host__ __device__ constexpr Plan half_plan() {
    return SPLIT ? make_split_plan(NT, RB, kHalfSB, 0, NT, 0) : make_plan(NT, RB, kHalfSB, 0, NT);
}
// Reals of its buffer.
__host__ __device__ constexpr int half_lds_reals(const Plan& P) {
    return P.nrounds < 2 ? 1 : (int)pad_rt((1u << P.tb) - 1u, kHalfSB) + 1;
}

// The order in which the plain transform of 2^N values butterflies its bits:
// on chip the top five, the low five, the rest upwards; above (FP32) pass 1's
// four top row bits of 12, its low four and the rest, then the column bits.
struct BitOrder {
    int bit[kMaxTileBits + 1] = {};
};
template <typename Real>
__host__ __device__ constexpr BitOrder plain_order(int N) {
    BitOrder o{};
    const bool two = N > Tune<Real>::FMAX;
    const int rows = two ? Tune<Real>::ROW : N, g = two ? Tune<Real>::RB1 : 5;
    int n = 0;
    for (int b = rows - g; b < rows; ++b) o.bit[n++] = b;
    for (int b = 0; b < rows - g; ++b) o.bit[n++] = b;
    for (int b = rows; b < N; ++b) o.bit[n++] = b;
    return o;
}
// Shift 0: element bit e of the half transform (its j-th butterfly) is bit
// plain_order[j] of k; the last of that order packs the halves into the real
// and imaginary part.
template <typename Real, int NT, int RB>
__host__ __device__ constexpr BitOrder zero_map() {
    constexpr Plan P = half_plan<NT, RB, 0>();
    constexpr BitOrder o = plain_order<Real>(NT + 1);
    BitOrder m{};
    int n = 0;
    for (int r = 0; r < P.nrounds; ++r)
        for (int b = 0; b < NT; ++b)
            if ((P.r[r].bfly >> b) & 1u) m.bit[b] = o.bit[n++];
    m.bit[NT] = o.bit[n];
    return m;
}

// Which set bit of x is left out (hb).  Any gives S_x.  HB_TOP: the top one.
// HB_LAST: the one the plain transform of 2^N values butterflies last (its
// order: the top five bits, the low five, the rest upwards).  With the others
// transformed in that same order, every later bit is clear in x, so the pair
// k, k ^ x meets element by element at its stage, whose results are exactly
// (2 Re, 0) and (0, 2 Im): the values keep every bit of the plain transform,
// which is what the counts of the plain forms' histogram depend on.
enum HalfBit { HB_TOP, HB_LAST };

// The left-out bit of a shift x != 0, and whether x has top bits only (HB_LAST).
struct HalfShift {
    uint32_t hb;
    bool top5;
};
template <bool HIST>
__host__ __device__ constexpr HalfShift half_shift(uint32_t x, int N, int bit) {
    uint32_t hb = 31u - (uint32_t)__builtin_clz(x);
    bool top5 = false;
    if constexpr (HIST) {
        const uint32_t mid = x & bits_range(5, N - 5), low = x & 31u;
        if (bit == HB_LAST && (mid | low)) hb = 31u - (uint32_t)__builtin_clz(mid ? mid : low);
        top5 = bit == HB_LAST && !(mid | low);
    }
    return HalfShift{hb, top5};
}
// Index k of element e: e with a zero inserted at bit hb.  Maps disjoint bits
// to disjoint bits.
template <bool HIST>
__host__ __device__ constexpr uint32_t half_k(uint32_t e, int N, const HalfShift& s) {
    if constexpr (HIST) {
        // x has top bits only: the first round keeps the other four and takes
        // bit 0 as its last
        if (s.top5)
            return ((e << 1) & bits_range(1, N - 5)) |
                   insert0(((e >> (N - 6)) & 15u) << (N - 5), s.hb) | (e >> (N - 2));
    }
    return insert0(e, s.hb);
}

}  // namespace sre2
