"""Half slabs of the two-pass kernels at sizes that take two passes (FP32 and split
forms from N = 17, FP64 from 16, SPLIT_BF16 from 15; smaller N run on chip):
the chunks of ragged shift ranges, the general index and the spectrum.

* Chunks: a range that starts inside a block of 2^L shifts, cut at a few shifts
  per launch and at the default, so that launches cross block edges (two values
  of x >> L, hence of the left-out row bit, in one launch).  Row pairs on and off
  agree bit for bit in the plain forms, and every chunking with the others.
* General index: of a product state A x B, sum_P |<P>|^(2 alpha) factors over
  the two parts, so M_alpha(A x B) = M_alpha(A) + M_alpha(B), both from the FP64
  oracle; A and B are Haar random and their qubits are dealt over rows and
  columns alike.  Bars of M_alpha: 1e-5 (FP32), 1e-9 (FP64).  Haar states: half slabs
  against full slabs within the same bars.
* Spectrum: counts of the half slabs equal to those of the full slabs."""
import functools

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_24685_amd as sre2  # noqa: E402

TOL_SX = {"fp32": 1e-4, "fp32h": 1e-4, "split16": 1e-4, "splitbf16": 1e-4,
          "fp64": 1e-11, "fp64h": 1e-11}
TOL_M = {"fp32": 1e-5, "fp32h": 1e-5, "fp64": 1e-9, "fp64h": 1e-9}
ALPHAS = (0.5, 1.0, 1.5, 3.0, 4.0)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(psi):
    return torch.from_numpy(np.ascontiguousarray(psi)).to("cuda")


def haar(N, seed, form):
    return W.haar(N, seed, np.complex128 if form.startswith("fp64") else np.complex64)


@pytest.fixture
def contexts():
    """(row pairs on, off), with launch counts."""
    on, off = sre2.Context(0), sre2.Context(0)
    off.set_row_pairs(False)
    for c in (on, off):
        c.set_timing(True)
    yield on, off
    on.close()
    off.close()


@pytest.mark.parametrize("form,N", [("fp32", 17), ("fp32", 18), ("fp32h", 17), ("fp64", 16),
                                    ("fp64", 17), ("fp64h", 16), ("split16", 17),
                                    ("splitbf16", 15), ("splitbf16", 16), ("splitbf16", 17)])
def test_chunks_across_block_edges(oracle_mod, contexts, form, N):
    psi_np = haar(N, 1611 + N, form)
    psi = dev(psi_np)
    L = sre2.row_bits(N, form)
    x0, xc = (1 << L) + 3, 2 * (1 << L) + 613
    print("CASE half slabs ragged", form, N, x0, xc, flush=True)
    on, off = contexts
    elem = 16 if form.startswith("fp64") else 8
    half = elem << (N - 1)  # bytes of one shift's half slab
    got = {}
    for name, ctx, slab in (("on", on, half), ("off", off, 2 * half)):
        if form.endswith("h"):
            slab = half
        for per in (8, 1 << L):
            ctx.set_scratch_limit(per * slab)
            got[name, per] = sre2.shift_partials(psi, x0, xc, form=form, ctx=ctx).cpu().numpy()
            assert ctx.timing_read()["pass1"][1] == -(-xc // per)  # a two-pass call, cut so
        assert np.array_equal(got[name, 8], got[name, 1 << L])
    a, b = got["on", 8], got["off", 8]
    if form.startswith("split"):
        assert np.max(np.abs(a - b) / b) <= TOL_SX[form]
    else:
        assert np.array_equal(a, b)
    edge = (1 << L) - 3  # first shift of the next block
    pick = np.array([0, 1, edge - 1, edge, edge + 4, edge + (1 << L), xc - 1])
    ref = oracle_mod.partials(psi_np, x0 + pick)
    assert np.max(np.abs(a[pick] - ref) / ref) <= TOL_SX[form]


@functools.lru_cache(maxsize=None)
def product_case(N, c128):
    """A x B on N qubits with A's qubits at the even positions (from the top
    as long as they last), and the exact M_alpha."""
    import oracle
    dt = np.complex128 if c128 else np.complex64
    na = (N + 1) // 2
    a, b = W.haar(na, 31 + N, np.complex128), W.haar(N - na, 32 + N, np.complex128)
    psi = np.kron(a, b).reshape((2,) * N)
    # axis i of kron -> position: A's at 0, 2, 4, ..., B's at 1, 3, ...
    order = np.argsort([2 * i for i in range(na)] + [2 * i + 1 for i in range(N - na)])
    psi = np.ascontiguousarray(psi.transpose(order)).reshape(-1).astype(dt)
    return psi, {al: oracle.sre(a, al) + oracle.sre(b, al) for al in ALPHAS}


@pytest.mark.parametrize("form,N", [("fp32", 17), ("fp32", 18), ("fp32h", 17), ("fp64", 16),
                                    ("fp64", 17), ("fp64h", 16)])
def test_general_index_of_product_states(oracle_mod, contexts, form, N):
    psi_np, want = product_case(N, form.startswith("fp64"))
    psi = dev(psi_np)
    for alpha in ALPHAS:
        for ctx in contexts:  # half slabs; full slabs
            print("CASE half slabs alpha", form, N, alpha, ctx is contexts[0], flush=True)
            r = sre2.sre(psi, alpha, form=form, ctx=ctx)
            assert r.status == 0 and ctx.timing_read()["pass1"][1] > 0
            assert abs(r.m2 - want[alpha]) <= TOL_M[form], (alpha, r.m2, want[alpha])


@pytest.mark.parametrize("form,N", [("fp32", 17), ("fp64", 16)])
def test_general_index_of_haar_states(contexts, form, N):
    psi = dev(haar(N, 1700 + N, form))
    for alpha in ALPHAS:
        print("CASE half slabs haar", form, N, alpha, flush=True)
        a, b = (sre2.sre(psi, alpha, form=form, ctx=c) for c in contexts)
        assert a.status == 0 and b.status == 0 and abs(a.m2 - b.m2) <= TOL_M[form], alpha


@pytest.mark.parametrize("form,N", [("fp32", 15), ("fp32", 16), ("fp32", 17), ("fp64", 16)])
def test_spectrum_counts_equal_full_slabs(contexts, form, N):
    """FP32: the half slabs keep every bit of the plain transform.  FP64: they do
    not, but of 2^32 strings about 10^-5 lie within a rounding of a bin edge."""
    psi = dev(haar(N, 1800 + N, form))
    print("CASE half slabs spectrum", form, N, flush=True)
    (a, _), (b, _) = (sre2.pauli_spectrum(psi, N + 8, form=form, ctx=c) for c in contexts)
    assert all(c.timing_read()["pass1"][1] > 0 for c in contexts)
    assert a.sum() == 4 ** N and np.array_equal(a, b)
