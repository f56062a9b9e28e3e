// sre2_both.h - last stage of a full slab whose two row halves were transformed
// apart (pass 2 with row pairs switched off), and the terms of its values.
// Host-compilable, so that the stage can be checked without a GPU.
#pragma once
#include <stdint.h>

namespace sre2 {

// Remove bit `b` of `v` (the bits above it move down by one): the inverse
// of insert0 on values with that bit clear.  Like insert0 it maps disjoint
// bit sets to disjoint bit sets, so it adds over them.
__host__ __device__ constexpr uint32_t remove_bit(uint32_t v, int b) {
    return ((v >> (b + 1)) << b) | (v & ((1u << b) - 1u));
}

__host__ __device__ constexpr uint32_t parity(uint32_t v) {
    return (uint32_t)__builtin_popcount(v) & 1u;
}

// x on the index bits of a column tile with row bit j left out: the row part
// xh without j above the tile's CB column bits, those of the column part xl.
__host__ __device__ constexpr uint32_t both_mask(uint32_t xh, uint32_t xl, int j, int CB) {
    return (remove_bit(xh, j) << CB) | (xl & ((1u << CB) - 1u));
}

// |v + u|^4 + |v - u|^4: the two values along the left-out row bit j, v and u
// being the transforms of the rows with j clear and set.  Both values count
// with both parts.  f_x(k ^ x) = conj f_x(k) makes u = s conj(v) with
//   s = (-1)^popcount(z & x), z the index of the values without bit j,
// so one value is real and the other imaginary: v + u where s = 1 (odd = 0), v - u
// where s = -1.  The square of the real one is the fused one, which is the order
// that the half slabs' 16 (Re^4 + Im^4) has: the sums agree bit for bit.
template <typename C>
__host__ __device__ inline double both_terms(C v, C u, uint32_t odd) {
    const auto px = v.x + u.x, py = v.y + u.y;
    const auto mx = v.x - u.x, my = v.y - u.y;
    const double p = (double)(px * px + py * py), m = (double)(mx * mx + my * my);
    const double re = odd ? m : p, im = odd ? p : m;
    return __builtin_fma(re, re, im * im);
}

}  // namespace sre2
