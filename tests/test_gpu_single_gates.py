"""Gates one call at a time (and a pass that is left with one gate) against the CPU
dynamics oracle: smallest sizes, neighbouring and far pairs in both orders, the pair
(0, 1), which keeps the tiles, and bits above a workgroup's 256 groups; bit for
bit what the same gates give in one call.

Tolerance: as for the gate passes, 1e-15 per gate on a state of norm 1: 1e-12."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_24685_amd as sre2  # noqa: E402
from oracle import dynamics as D  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N", [2, 3, 9, 10, 11, 13, 15])
def test_one_gate_per_call(N):
    rng = np.random.default_rng(900 + N)
    pairs = {(0, 1), (1, 0), (N - 1, N - 2), (0, N - 1), (N - 1, 0), (N // 2, N // 2 - 1)}
    pairs |= {tuple(int(q) for q in rng.choice(N, 2, replace=False)) for _ in range(6)}
    pairs = sorted(p for p in pairs if p[0] != p[1])
    gates = [W.haar_u4(rng) for _ in pairs]
    th, ph = W.product_angles(N, 60 + N)
    print("CASE single gates", N, pairs, flush=True)
    sim, once = sre2.Simulator(N), sre2.Simulator(N)
    ref = D.product_state(th, ph)
    for s in (sim, once):
        s.product_state(th, ph)
    for U, (a, b) in zip(gates, pairs):
        sim.apply_gates([U], [(a, b)])
        ref = D.apply_2q(ref, U, a, b)
    once.apply_gates(gates, pairs)
    got = sim.state()
    assert np.abs(got.cpu().numpy() - ref).max() < 1e-12
    assert torch.equal(got, once.state())
    for s in (sim, once):
        s.close()
