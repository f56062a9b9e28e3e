"""Gate passes of the simulator (several gates per tile of 11 qubits) against
the CPU dynamics oracle: sizes below, at and above the tile, more gates than
one pass holds and than the planner looks ahead, pairs in any order.

Tolerance: each gate is a unitary on four amplitudes, whose rounding adds at
most about 1e-15 to a state of norm 1 per gate; 300 gates stay below 1e-12."""
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


@pytest.mark.parametrize("N,count", [(2, 3), (3, 16), (4, 15), (10, 40), (11, 14), (12, 300),
                                     (14, 31), (15, 2)])
def test_random_pairs_match_oracle(N, count):
    rng = np.random.default_rng(100 * N + count)
    pairs = [tuple(int(q) for q in rng.choice(N, 2, replace=False)) for _ in range(count)]
    gates = [W.haar_u4(rng) for _ in range(count)]
    th, ph = W.product_angles(N, 60 + N)
    print("CASE gate passes", N, count, flush=True)
    sim = sre2.Simulator(N)
    sim.product_state(th, ph)
    ref = D.product_state(th, ph)
    assert np.abs(sim.state().cpu().numpy() - ref).max() < 1e-15
    sim.apply_gates(gates, pairs)
    for U, (a, b) in zip(gates, pairs):
        ref = D.apply_2q(ref, U, a, b)
    assert np.abs(sim.state().cpu().numpy() - ref).max() < 1e-12
    sim.close()
