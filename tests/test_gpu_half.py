"""The on-chip half transforms (k_half) at the edges of their range, against
the FP64 CPU oracle: ranges that are shift 0 alone, start or end at it, or
hold the last shifts; the smallest and largest N per precision, and the FP16
split form, whose shift 0 takes another kernel (k_fused up to N = 14, two-pass
above); and the BF16 form's rebuilt rows (k_pass2_images) with the left-out row
bit in a register and in the thread index.

Tolerances: an S_x is a sum of 2^N fourth powers whose values carry the
rounding of N - 1 additions each (relative to the largest |W|, which is n at
shift 0): the per-shift bars of the two precisions, 1e-4 (FP32) and 1e-11
(FP64); the general index keeps the bars of M_alpha, 1e-5 and 1e-9."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_24685_amd as sre2  # noqa: E402

TOL_SX = {"fp32": 1e-4, "fp32h": 1e-4, "split16": 1e-4, "splitbf16": 1e-4,
          "fp64": 1e-11, "fp64h": 1e-11}


def dev(psi):
    return torch.from_numpy(np.ascontiguousarray(psi)).to("cuda")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("form,N", [("fp32", 10), ("fp32", 11), ("fp32", 12), ("fp32", 14),
                                    ("fp32", 15), ("fp32", 16), ("fp32h", 16),
                                    ("split16", 13), ("split16", 14), ("split16", 15),
                                    ("split16", 16), ("splitbf16", 15),
                                    ("splitbf16", 16), ("fp64", 10), ("fp64", 11), ("fp64", 13),
                                    ("fp64", 14), ("fp64h", 15)])
def test_range_edges(oracle_mod, form, N):
    c128 = form.startswith("fp64")
    psi = W.haar(N, 4200 + N, np.complex128 if c128 else np.complex64)
    d = dev(psi)
    D = 1 << N
    for x0, xc in ((0, 1), (0, 3), (1, 1), (D // 2 - 1, 3), (D - 2, 2)):
        print("CASE half", form, N, x0, xc, flush=True)
        got = sre2.shift_partials(d, x0, xc, form=form).cpu().numpy()
        ref = oracle_mod.partials(psi, np.arange(x0, x0 + xc))
        assert got.shape == (xc,)
        assert np.max(np.abs(got - ref) / ref) <= TOL_SX[form], (x0, xc)


@pytest.mark.parametrize("form,N", [("fp32", 12), ("fp32", 15), ("fp64", 11), ("fp64", 14)])
@pytest.mark.parametrize("alpha", [0.5, 1.0, 3.0])
def test_general_index(oracle_mod, form, N, alpha):
    """|T>^N (every value a product of 1 and 2^-1/2): the closed form
    M_alpha = N log2((1 + 2^(1 - alpha)) / 2) / (1 - alpha), N / 2 at 1."""
    c128 = form.startswith("fp64")
    d = dev(W.t_product(N, np.complex128 if c128 else np.complex64))
    print("CASE half alpha", form, N, alpha, flush=True)
    r = sre2.sre(d, alpha, form=form)
    ref = N / 2 if alpha == 1.0 else N * np.log2((1 + 2.0 ** (1 - alpha)) / 2) / (1 - alpha)
    assert r.status == 0 and abs(r.m2 - ref) <= (1e-9 if c128 else 1e-5)


@pytest.mark.parametrize("form,N", [("fp32", 5), ("fp32", 10), ("fp32", 12), ("fp32", 14),
                                    ("split16", 13), ("fp64", 11), ("fp64", 13)])
def test_packed_states_equal_single_calls(form, N):
    c128 = form.startswith("fp64")
    psis = [dev(W.haar(N, 4300 + j, np.complex128 if c128 else np.complex64)) for j in range(3)]
    print("CASE half packed", form, N, flush=True)
    for p, b in zip(psis, sre2.m2_batched(psis, form=form)):
        a = sre2.m2(p, form=form, partials=True)
        assert a.m2 == b.m2 and a.S == b.S and b.status == 0
        # the end of the evaluation: sum of S_x and the norm, in FP64
        assert abs(a.S - a.partials.sum().item()) <= 1e-14 * a.S
        assert abs(a.n - 1.0) <= (1e-13 if c128 else 1e-6)
        c = sre2.m2_from_partials(p, a.partials, form=form)
        assert a.m2 == c.m2 and a.n == c.n


@pytest.mark.parametrize("form,N", [("fp32", 12), ("fp32", 14), ("fp32", 15), ("fp32", 17),
                                    ("fp32h", 13), ("fp64", 11), ("fp64", 15)])
def test_spectrum_counts_are_the_plain_transforms(oracle_mod, form, N):
    """Every shift of |T>^N has its values at 0 and n 2^-popcount(...): exact
    counts C(N, k) 2^k whichever bit a half transform leaves out (shift 0, the
    shifts of the top five bits, low bits, middle bits); a Haar state's counts
    against the oracle, up to the strings near a bin edge."""
    from math import comb
    c128 = form.startswith("fp64")
    dt = np.complex128 if c128 else np.complex64
    print("CASE half spectrum", form, N, flush=True)
    counts, _ = sre2.pauli_spectrum(dev(W.t_product(N, dt)), N + 3, form=form)
    for k in range(N + 1):
        assert counts[k] == comb(N, k) * 2 ** k
    assert counts.sum() == 4 ** N
    if N <= 14:
        psi = W.haar(N, 4400 + N, dt)
        counts, _ = sre2.pauli_spectrum(dev(psi), N + 6, form=form)
        ref, near = oracle_mod.spectrum(psi, N + 6, eps=2e-3 if not c128 else 1e-7)
        assert int(np.abs(counts - ref).sum()) <= 2 * near
