// sre2_twopass.h - slab geometry shared by the two passes of the transforms
// above the on-chip range.
#pragma once
#include "sre2_tile.h"

namespace sre2 {

// Slab geometry of a two-pass slab kind: slab bits NS of one shift and
// pass-1 row bits L (the row pairs keep the rows and columns of the full
// slab and store half its rows).
template <typename Real>
void slab_geometry(int N, int slab, int* NS, int* L) {
    *NS = N - (slab == kSlabHerm || slab == kSlabPairs ? 1 : 0);
    *L = row_bits_of<Real>(slab == kSlabHerm ? N - 1 : N);
}

}  // namespace sre2
