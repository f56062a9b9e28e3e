// Host-only probe of the on-chip half transforms' plans and index maps
// (sre2_half_map.h, sre2_geometry.h), compiled with g++ by tests/test_half_plan.py.
#include <utility>
#define __host__
#define __device__
#include "../paper_2512_24685_amd/csrc/sre2_half_map.h"

namespace {
using namespace sre2;

// kind 0: M2 and general sums, 1: histogram, 2: FP16 split form
constexpr int kM2 = 0, kHist = 1, kSplit = 2;
template <typename Real>
bool range(int kind, int* lo, int* hi) {
    using T = Tune<Real>;
    if (kind == kSplit && sizeof(Real) == 8) return false;
    *lo = kind == kSplit ? T::HSPLIT : kind == kHist ? half_hist_min<Real>() : T::HMIN;
    *hi = kind == kHist ? half_hist_max<Real>() : T::HMAX;
    return true;
}

struct Info {
    Plan p;
    BitOrder zero;
    int reals;
};
template <typename Real, int N>
Info info_of(int kind) {
    constexpr int RBM = half_rb<Real>(N, false), RBH = half_rb<Real>(N, true);
    Info i{};
    if (kind == kM2) {
        i.p = half_plan<N - 1, RBM, 0>();
        i.zero = zero_map<Real, N - 1, RBM>();
    } else if (kind == kHist) {
        if constexpr (N >= half_hist_min<Real>()) {
            i.p = half_plan<N - 1, RBH, 0>();
            i.zero = zero_map<Real, N - 1, RBH>();
        }
    } else if constexpr (sizeof(Real) == 4 && N >= Tune<Real>::HSPLIT) {
        i.p = half_plan<N - 1, RBH, 1>();
    }
    i.reals = half_lds_reals(i.p);
    return i;
}
template <typename Real, int... Ns>
Info info(int N, int kind, std::integer_sequence<int, Ns...>) {
    Info r{};
    ((N == Ns + Tune<Real>::HMIN ? (r = info_of<Real, Ns + Tune<Real>::HMIN>(kind), 0) : 0), ...);
    return r;
}
Info info(int precision, int N, int kind) {
    return precision == 0
               ? info<float>(N, kind,
                             std::make_integer_sequence<int, Tune<float>::HMAX - Tune<float>::HMIN + 1>{})
               : info<double>(N, kind,
                              std::make_integer_sequence<int, Tune<double>::HMAX - Tune<double>::HMIN + 1>{});
}
}  // namespace

extern "C" {

// Smallest and largest N of a kind; -1 where the precision has none.
int probe_range(int precision, int kind, int* lo, int* hi) {
    return (precision == 0 ? range<float>(kind, lo, hi) : range<double>(kind, lo, hi)) ? 0 : -1;
}

// Rounds (reg, bfly, lane, wave, lperm, mf), register bits, reals of the
// buffer, and shift 0's bit map (N entries); returns the round count.
int probe_half(int precision, int N, int kind, unsigned* out, int* rb, int* reals, int* zero) {
    const Info i = info(precision, N, kind);
    for (int j = 0; j < i.p.nrounds; ++j) {
        const Round& r = i.p.r[j];
        const unsigned w[6] = {r.reg, r.bfly, r.lane, r.wave, r.lperm, r.mf};
        for (int q = 0; q < 6; ++q) out[6 * j + q] = w[q];
    }
    for (int b = 0; b < N; ++b) zero[b] = i.zero.bit[b];
    *rb = i.p.rb;
    *reals = i.reals;
    return i.p.nrounds;
}

// Left-out bit and k of every element of shift x.
int probe_map(int N, unsigned x, int hist, int last, unsigned* k) {
    const int bit = last ? HB_LAST : HB_TOP;
    const HalfShift s = hist ? half_shift<true>(x, N, bit) : half_shift<false>(x, N, bit);
    for (unsigned e = 0; e < 1u << (N - 1); ++e)
        k[e] = hist ? half_k<true>(e, N, s) : half_k<false>(e, N, s);
    return (int)s.hb;
}

void probe_plain_order(int precision, int N, int* out) {
    const BitOrder o = precision == 0 ? plain_order<float>(N) : plain_order<double>(N);
    for (int b = 0; b < N; ++b) out[b] = o.bit[b];
}
unsigned probe_slot(unsigned e) { return pad16<kHalfSB>(e); }
}
