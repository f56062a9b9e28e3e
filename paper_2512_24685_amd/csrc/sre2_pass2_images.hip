// sre2_pass2_images.hip - pass 2 of the BF16 split form at N = 15 and 16: full
// column transforms on rebuilt rows.
//
// Slab row r ^ xh of a shift x (xh = x >> L, xl = x mod 2^L) is the image
//   row(r ^ xh)[z] = (-1)^popcount(z & xl) conj(row(r)[z])
// of row r, so pass 1 stores only the rows with bit j = half_row_bit(xh,
// images_rows) clear, and this kernel rebuilds the others by sign flips.  The
// other forms transform the stored rows alone (k_pass2, HALF_SLAB; on chip,
// k_half), which gives the same values up to rounding at half the work.  With
// 16 significant bits that rounding would move the S_x of N = 15 and 16 by 2 to 4e-9
// (2-norm, shift 0 among them).  That is far inside the form's error bar, but
// sre2.h says that these sizes keep the bits of the rebuilt rows; from N = 17
// on, where S_x average over more values (6.5e-10), the BF16 form takes the
// half slabs too.
//
// j is taken among the register row bits when xh has one, so that which
// elements are rebuilt is fixed per register index (pair_load_reg); otherwise
// xh has only thread row bits and whole threads hold rebuilt rows
// (pair_load_thr).  Stored values are read twice inside one tile, the second
// time from the caches.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sre2_both.h"
#include "sre2_twopass.h"

namespace sre2 {

namespace {

// Flip the sign bits of a complex value's parts by the masks mx, my (each
// 0 or the sign bit of a float, applied to the high word of a double).
constexpr uint32_t kSign = 0x80000000u;
__device__ __forceinline__ float2 xor_signs(float2 v, uint32_t mx, uint32_t my) {
    v.x = __uint_as_float(__float_as_uint(v.x) ^ mx);
    v.y = __uint_as_float(__float_as_uint(v.y) ^ my);
    return v;
}

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

// Block b -> shift slot b / P, column group b % P, as in k_pass2; the next
// column tile is loaded while one is transformed.
template <int HT>
__global__ __launch_bounds__(1 << (pass2_tb<float>(HT) - Tune<float>::RB2))
__attribute__((amdgpu_waves_per_eu(SRE2_P2S_WAVES)))
void k_pass2_images(const float2* __restrict__ scratch, int N, int P, double* __restrict__ part,
                    const int* __restrict__ scale_exp, int64_t x0) {
    using C = float2;
    constexpr int TB = pass2_tb<float>(HT), RB = Tune<float>::RB2, SPLIT = 2;
    constexpr int T = 1 << (TB - RB);
    constexpr int PK = 3000 + HT + 10000 * SPLIT;
    constexpr Plan PL = plan_of<float, TB, RB, PK>();
    constexpr Round r0 = PL.r[0];
    constexpr int CB = TB - HT;  // column bits per tile
    constexpr uint32_t CMASK = (1u << CB) - 1u, RROW = r0.reg >> CB;
    static_assert(TB <= 12, "two register sets");
    __shared__ C lds[lds_values(PL)];
    __shared__ double red[T];
    const int64_t b = blockIdx.x;
    const int64_t s = b / P;
    const int g = (int)(b % P);
    const int L = N - HT;             // row bits of pass 1
    const int per = (1 << (L - CB)) / P;
    const int SH = N - 1;             // slab bits of one shift
    const auto rs = buf_rsrc(scratch + ((uint64_t)s << SH), (uint32_t)sizeof(C) << SH);
    // the shift's row and column parts, the left-out row bit, the thread's
    // stored-row (vb0) and partner-row (vb1) address parts and the sign
    // (-1)^popcount(z & xl) of its column bits
    const uint32_t base = thread_base<r0.lperm, r0.wave>();
    const uint64_t x = (uint64_t)(x0 + s);
    const uint32_t xh = (uint32_t)(x >> L), xl = (uint32_t)x & ((1u << L) - 1u);
    const int j = half_row_bit(xh, RROW);
    const uint32_t rowT = base >> CB, colT = base & CMASK;
    const uint32_t vb0 = (remove_bit(rowT, j) << L) + colT;
    const uint32_t vb1 = (remove_bit(rowT ^ (xh & ~RROW), j) << L) + colT;
    const uint32_t sT = __builtin_popcount(colT & xl) & 1u;
    const uint32_t fm = 0u - ((rowT >> j) & 1u);
    double acc = 0.0;
    auto consume = [&](C (&v)[1 << RB]) {
        run_transform<float, TB, RB, PK>(lds, v);
#pragma unroll
        for (int i = 0; i < (1 << RB); ++i) acc += abs4(v[i]);
    };
    const int c0 = g * per, c1 = (g + 1) * per;
    auto tiles = [&](auto&& load_tile) {
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
    };
    if ((RROW >> j) & 1u) {
        with_reg_row_bit<RROW>(j, [&](auto J) {
            tiles([&](C (&v)[1 << RB], int ct) {
                constexpr int JJ = decltype(J)::value;
                const uint32_t cto = (uint32_t)ct << CB;
                const uint32_t mT = ((sT ^ __builtin_popcount(cto & xl)) & 1u) ? kSign : 0u;
                pair_load_reg<C, RB, r0.reg, CB, JJ>(v, rs, L, vb0, vb1, xh, xl, cto, mT);
            });
        });
    } else {
        const uint32_t vbt = fm ? vb1 : vb0;
        tiles([&](C (&v)[1 << RB], int ct) {
            const uint32_t cto = (uint32_t)ct << CB;
            const uint32_t mT = ((sT ^ __builtin_popcount(cto & xl)) & 1u) ? kSign : 0u;
            pair_load_thr<C, RB, r0.reg, CB>(j, v, rs, L, vbt, fm, xl, cto, mT);
        });
    }
    acc *= ldexp(1.0, -4 * *scale_exp);
    const double tot = block_sum<T>(acc, red);
    if (threadIdx.x == 0) part[b] = tot;
}

template <int HT>
constexpr uint32_t images_rows_of() {
    constexpr int TB = pass2_tb<float>(HT);
    return plan_of<float, TB, Tune<float>::RB2, 3000 + HT + 20000>().r[0].reg >> (TB - HT);
}

}  // namespace

static_assert(kImagesMaxN - Tune<float>::ROW == 4, "row bits 3 (N = 15) and 4 (N = 16)");

uint32_t images_rows(int N) {
    return N - row_bits_of<float>(N) == 3 ? images_rows_of<3>() : images_rows_of<4>();
}

hipError_t launch_pass2_images(const void* scratch, int N, int64_t x0, int cs, int P,
                               double* part, const int* se, hipStream_t st) {
    const int HT = N - row_bits_of<float>(N);
    const dim3 grid((unsigned)((int64_t)cs * P));
    if (HT == 3)
        k_pass2_images<3><<<grid, 1 << (pass2_tb<float>(3) - Tune<float>::RB2), 0, st>>>(
            (const float2*)scratch, N, P, part, se, x0);
    else if (HT == 4)
        k_pass2_images<4><<<grid, 1 << (pass2_tb<float>(4) - Tune<float>::RB2), 0, st>>>(
            (const float2*)scratch, N, P, part, se, x0);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sre2
