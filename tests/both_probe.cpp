// Host-only probe of the last stage of a full slab transformed in two halves
// (sre2_both.h), compiled with g++ by tests/test_both_halves.py.
#define __host__
#define __device__
#include "../paper_2512_24685_amd/csrc/sre2_both.h"

namespace {
struct F2 {
    float x, y;
};
}  // namespace

extern "C" {
unsigned probe_mask(unsigned xh, unsigned xl, int j, int cb) {
    return sre2::both_mask(xh, xl, j, cb);
}
unsigned probe_parity(unsigned v) { return sre2::parity(v); }
// v, u: complex64 arrays of n values; out[i] = the terms of element i.
void probe_terms(const float* v, const float* u, const unsigned* odd, int n, double* out) {
    for (int i = 0; i < n; ++i)
        out[i] = sre2::both_terms(F2{v[2 * i], v[2 * i + 1]}, F2{u[2 * i], u[2 * i + 1]}, odd[i]);
}
}
