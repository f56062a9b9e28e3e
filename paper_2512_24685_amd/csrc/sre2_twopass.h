// sre2_twopass.h - slab geometry shared by the two passes of the transforms
// above the on-chip range.
#pragma once
#include <utility>

#include "sre2_tile.h"

namespace sre2 {

// Register row bits of the first round of the pass-2 tile of HT rows (split
// form s: its matrix-core plan): the preferred left-out row bits of the row
// pairs, so that pass 1 leaves out the rows pass 2 rebuilds.
template <typename Real, int HT, int SPLIT>
constexpr uint32_t pass2_reg_rows() {
    constexpr int TB = pass2_tb<Real>(HT), RB = Tune<Real>::RB2;
    return plan_of<Real, TB, RB, 3000 + HT + 10000 * SPLIT>().r[0].reg >> (TB - HT);
}
template <typename Real, int... Hs>
uint32_t pair_pref_of(int HT, int split, std::integer_sequence<int, Hs...>) {
    uint32_t m = 0;
    ((HT == Hs + 1 ? (m = split == 0 ? pass2_reg_rows<Real, Hs + 1, 0>()
                        : split == 1 ? pass2_reg_rows<Real, Hs + 1, 1>()
                                     : pass2_reg_rows<Real, Hs + 1, 2>(),
                      0)
                   : 0),
     ...);
    return m;
}

// Slab geometry of a two-pass slab kind: slab bits NS of one shift and
// pass-1 row bits L (the row pairs keep the rows and columns of the full
// slab and store half its rows).
template <typename Real>
void slab_geometry(int N, int slab, int* NS, int* L) {
    *NS = N - (slab == kSlabFull ? 0 : 1);
    *L = row_bits_of<Real>(slab == kSlabHerm ? N - 1 : N);
}

}  // namespace sre2
