"""TFIM steps against exact states at sizes above the CPU oracle's reach: the
workgroups of four (from N = 18) and two runs (from N = 22) of the Chebyshev term.

* J = 0: every qubit rotates by itself, exp(i dt (hx X + hz Z)), so a product
  state stays one.  A flip that is missing, doubled or of another bit, or a wrong
  longitudinal field, moves some amplitude by O(dt).
* hx = 0: the step multiplies amplitude k by exp(i dt (J sum s_i s_i+1 + hz sum s_i)),
  which fixes the diagonal.

H is the sum of these parts, each amplitude's row of it linear in (J, hx, hz); a step
with all of them is undone by its opposite in test_gpu_tfim_terms.py.

Tolerance: amplitudes are at most 1; up to 40 terms of about 1e-15 each, and the
reference's N complex factors of 1e-16 each: 1e-12."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_24685_amd as sre2  # noqa: E402

SIZES = [12, 17] + list(range(18, 27))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def product(cols):
    """Product state, qubit i (bit i) in the two amplitudes cols[i]."""
    psi = torch.ones(1, dtype=torch.complex128, device="cuda")
    for c in cols:
        psi = (torch.from_numpy(np.asarray(c, np.complex128)).cuda()[:, None] *
               psi[None, :]).reshape(-1)
    return psi


def stepped(N, J, hx, hz, dt):
    th, ph = W.product_angles(N, 170 + N)
    sim = sre2.Simulator(N)
    try:
        sim.product_state(th, ph)
        sim.tfim_step(J, hx, hz, dt)
        cols = [(np.cos(t / 2), np.exp(1j * p) * np.sin(t / 2)) for t, p in zip(th, ph)]
        return sim.state(), cols
    finally:
        sim.close()


@pytest.mark.parametrize("N", SIZES)
def test_field_alone_rotates_each_qubit(N):
    hx, hz, dt = 1.1, -0.6, 0.3
    print("CASE tfim exact field", N, flush=True)
    got, cols = stepped(N, 0.0, hx, hz, dt)
    h = np.hypot(hx, hz)
    c, s = np.cos(h * dt), 1j * np.sin(h * dt) / h
    R = np.array([[c + s * hz, s * hx], [s * hx, c - s * hz]])
    ref = product([R @ np.array(q) for q in cols])
    assert float((got - ref).abs().max()) < 1e-12


@pytest.mark.parametrize("N", SIZES)
def test_no_transverse_field_is_a_phase(N):
    J, hz, dt = 0.8, 0.35, 0.3
    print("CASE tfim exact phase", N, flush=True)
    got, cols = stepped(N, J, 0.0, hz, dt)
    k = torch.arange(1 << N, device="cuda")
    energy = torch.zeros(1 << N, dtype=torch.float64, device="cuda")
    s = 1.0 - 2.0 * (k & 1).double()
    for i in range(N):
        energy += hz * s
        if i + 1 < N:
            t = 1.0 - 2.0 * ((k >> (i + 1)) & 1).double()
            energy += J * s * t
            s = t
    ref = product(cols) * torch.polar(torch.ones_like(energy), dt * energy)
    assert float((got - ref).abs().max()) < 1e-12
