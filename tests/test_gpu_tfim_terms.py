"""Chebyshev steps of the simulator at the edges of their kernels, against the
CPU dynamics oracle (expm_multiply): the single-workgroup range (up to N = 11,
128 terms a launch), the sizes above it, both signs of the step, a step with
more terms than one launch holds, no field along x.

Tolerance: the series is cut below 1e-17 and its terms T_k of norm at most 1
carry about 1e-15 each in FP64, up to 300 of them here; with the oracle's own error
1e-11, the bar of the other step tests.  Above the oracle's reach (N = 18, 19:
four runs per workgroup) the step is undone by the opposite one, to 1e-12."""
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


@pytest.mark.parametrize("N,J,hx,hz,dt", [(2, 1.0, 1.5, 1.5, 0.2), (5, -0.7, 0.4, -1.1, -0.3),
                                          (9, 1.0, 1.5, 1.5, 6.0), (10, 1.0, 0.0, 0.5, 0.4),
                                          (11, 1.0, 1.5, 1.5, 0.2), (12, 1.0, 1.5, 1.5, -0.2),
                                          (13, 0.3, -2.0, 0.1, 0.5)])
def test_step_matches_oracle(N, J, hx, hz, dt):
    th, ph = W.product_angles(N, 70 + N)
    print("CASE tfim terms", N, dt, flush=True)
    sim = sre2.Simulator(N)
    sim.product_state(th, ph)
    sim.tfim_step(J, hx, hz, dt)
    H = D.tfim_hamiltonian(N, J, hx, hz)
    ref = D.tfim_evolve(D.product_state(th, ph), H, dt)
    assert np.abs(sim.state().cpu().numpy() - ref).max() < 1e-11
    sim.close()


@pytest.mark.parametrize("N", [17, 18, 19])
def test_step_back_undoes_step(N):
    th, ph = W.product_angles(N, 70 + N)
    print("CASE tfim back", N, flush=True)
    sim = sre2.Simulator(N)
    sim.product_state(th, ph)
    a = sim.state()
    sim.tfim_step(1.0, 1.5, 1.5, 0.2)
    b = sim.state()
    assert float((b - a).abs().max()) > 1e-6  # the step moves the state
    sim.tfim_step(1.0, 1.5, 1.5, -0.2)
    assert float((sim.state() - a).abs().max()) < 1e-12
    sim.close()
