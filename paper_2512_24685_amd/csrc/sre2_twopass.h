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
    *NS = N - (slab == kSlabHerm || slab == kSlabPairs || slab == kSlabImages ? 1 : 0);
    *L = row_bits_of<Real>(slab == kSlabHerm ? N - 1 : N);
}

// Pass 2 on rebuilt rows (kSlabImages), and the row bits pass 1 leaves out by
// preference for it: those the pass-2 plan holds in registers.
hipError_t launch_pass2_images(const void* scratch, int N, int64_t x0, int cs, int P,
                               double* part, const int* se, hipStream_t st);
uint32_t images_rows(int N);

}  // namespace sre2
