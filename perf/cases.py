"""Performance cases: what users of this package have it compute, over the
sizes, element types, arithmetic forms and options they use.

A case is a dict of plain values; ``prepare`` makes the device state (or the
simulator) a user's program holds before the call, ``run`` makes the call.
States are Haar random, the ensemble the XOR-FWHT method is benchmarked on;
the dynamics cases start from random product states.

Kinds
  m2        one state, every Pauli string (m2_async); optionally with S_x
  batch     many small states in one call (m2_batched), as a serving loop packs
  sre       general Renyi index
  spectrum  Pauli-spectrum histogram
  shard     S_x of a leading range of shifts (rank 0 of a sharded evaluation)
  tfim      Hamiltonian quench: product state, Chebyshev steps, state read out
  circuit   brickwork circuit: product state, gate layers, state read out
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2512_24685_amd as sre2

C64, C128 = "complex64", "complex128"
FORMS32 = ("fp32", "fp32h", "split16", "splitbf16")
FORMS64 = ("fp64", "fp64h")


def listed():
    return [
        # a single small state in double precision: launches and latency
        {"name": "m2_n10_c128_fp64", "kind": "m2", "N": 10, "dtype": C128, "form": "fp64",
         "partials": False},
        # small requests of a serving stream (N from 8 up), packed by N
        {"name": "batch48_n8_12_fp32", "kind": "batch", "count": 48, "N_min": 8, "N_max": 12,
         "dtype": C64, "form": "fp32"},
        # ordinary state in double precision, on chip
        {"name": "m2_n13_c128_fp64", "kind": "m2", "N": 13, "dtype": C128, "form": "fp64",
         "partials": False},
        # ordinary state, every S_x kept
        {"name": "m2_n14_fp32_sx", "kind": "m2", "N": 14, "dtype": C64, "form": "fp32",
         "partials": True},
        # Pauli spectrum of an ordinary state
        {"name": "spectrum_n13_fp32", "kind": "spectrum", "N": 13, "dtype": C64, "form": "fp32",
         "nbins": 32},
        # third Renyi index, first size of the two-pass path
        {"name": "sre3_n15_fp32", "kind": "sre", "N": 15, "dtype": C64, "form": "fp32",
         "alpha": 3.0},
        # the size of the 40-state batch workload, in single precision and in
        # the double-precision Hermitian pair
        {"name": "m2_n16_fp32", "kind": "m2", "N": 16, "dtype": C64, "form": "fp32",
         "partials": False},
        {"name": "m2_n16_c128_fp64h", "kind": "m2", "N": 16, "dtype": C128, "form": "fp64h",
         "partials": False},
        # the largest request of the serving stream, on the matrix cores
        {"name": "m2_n18_split16", "kind": "m2", "N": 18, "dtype": C64, "form": "split16",
         "partials": False},
        # the throughput workload's state, a quarter of its shifts (four ranks)
        {"name": "shard_n20_fp32", "kind": "shard", "N": 20, "dtype": C64, "form": "fp32",
         "x_count": 1 << 18},
        # quench dynamics: TFIM steps at the snapshot pipeline's size, and a
        # large brickwork circuit
        {"name": "tfim_n16", "kind": "tfim", "N": 16, "steps": 2},
        {"name": "circuit_n20", "kind": "circuit", "N": 20, "layers": 4},
    ]


def draw(rng):
    kind = rng.choice(("m2", "m2", "m2", "m2", "batch", "spectrum", "sre", "shard", "tfim",
                       "circuit"))
    if kind == "tfim":
        return {"kind": kind, "N": rng.randint(6, 19), "steps": rng.randint(1, 3)}
    if kind == "circuit":
        return {"kind": kind, "N": rng.randint(6, 22), "layers": rng.randint(1, 6)}
    double = rng.random() < 0.4
    c = {"kind": kind, "dtype": C128 if double or rng.random() < 0.1 else C64}
    if kind == "m2":
        c["form"] = rng.choice(FORMS64 if double else FORMS32 + ("fp32",))
        c["N"] = rng.randint(6, 17 if double else 18)
        c["partials"] = c["N"] >= 13 and rng.random() < 0.3
    elif kind == "batch":
        c["form"] = rng.choice(FORMS64 if double else FORMS32)
        c["count"] = int(round(math.exp(rng.uniform(math.log(3), math.log(90)))))
        c["N_min"] = rng.randint(6, 10)
        c["N_max"] = c["N_min"] + rng.randint(0, 4)
    elif kind == "spectrum":
        c["form"] = rng.choice(FORMS64 if double else ("fp32", "fp32h"))
        c["N"] = rng.randint(7, 15)
        c["nbins"] = rng.randint(12, 64)
    elif kind == "sre":
        c["form"] = rng.choice(FORMS64 if double else ("fp32", "fp32h"))
        c["N"] = rng.randint(7, 16)
        c["alpha"] = rng.choice((0.5, 1.0, 1.5, 3.0, 4.0))
    else:
        # the start of the shift range, ragged lengths
        c["form"] = rng.choice(FORMS64 if double else FORMS32)
        c["N"] = rng.randint(18, 21)
        c["x_count"] = int(math.exp(rng.uniform(math.log(1 << 9), math.log(1 << 15)))) | 1
    return c


def _haar(N, dtype, gen):
    psi = torch.randn(1 << N, dtype=torch.complex128, device="cuda", generator=gen)
    psi /= torch.linalg.vector_norm(psi)
    return psi.to(getattr(torch, dtype))


def _batch_sizes(case):
    span = case["N_max"] - case["N_min"] + 1
    return [case["N_min"] + i % span for i in range(case["count"])]


def _haar_u4(count, rng):
    a = rng.standard_normal((count, 4, 4)) + 1j * rng.standard_normal((count, 4, 4))
    q, r = np.linalg.qr(a)
    d = np.diagonal(r, axis1=1, axis2=2)
    return q * (d / np.abs(d))[:, None, :]


TFIM = (1.0, 1.5, 1.5, 0.2)  # J, hx, hz, dt


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("tfim", "circuit"):
        N = case["N"]
        rng = np.random.default_rng(seed)
        st = {"case": case, "sim": sre2.Simulator(N), "theta": rng.uniform(0.0, np.pi, N),
              "phi": rng.uniform(0.0, 2.0 * np.pi, N)}
        if kind == "circuit":
            bonds = [(i, i + 1) for i in range(0, N - 1, 2)] + [(i, i + 1)
                                                                for i in range(1, N - 1, 2)]
            st["pairs"] = np.array(bonds * case["layers"], dtype=np.int32)
            st["gates"] = _haar_u4(len(st["pairs"]), rng)
        return st
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "batch":
        return {"case": case, "psi": [_haar(N, case["dtype"], gen) for N in _batch_sizes(case)]}
    return {"case": case, "psi": _haar(case["N"], case["dtype"], gen)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "m2":
        out, part = sre2.m2_async(state["psi"], case["form"], partials=case["partials"])
        return (out, part) if case["partials"] else (out,)
    if kind == "batch":
        res = sre2.m2_batched(state["psi"], case["form"])
        return np.array([(r.m2, r.S, r.n, r.status) for r in res])
    if kind == "sre":
        r = sre2.sre(state["psi"], case["alpha"], case["form"])
        return np.array([r.m2, r.S, r.n])
    if kind == "spectrum":
        counts, r = sre2.pauli_spectrum(state["psi"], case["nbins"], case["form"])
        return {"counts": counts, "n": r.n}
    if kind == "shard":
        return sre2.shift_partials(state["psi"], 0, case["x_count"], case["form"])
    sim = state["sim"]
    sim.product_state(state["theta"], state["phi"])
    if kind == "tfim":
        for _ in range(case["steps"]):
            sim.tfim_step(*TFIM)
    else:
        sim.apply_gates(state["gates"], state["pairs"])
    return sim.state()


def work(case):
    kind = case["kind"]
    if kind in ("tfim", "circuit"):
        # angles (and gates) in, the state out; per amplitude and qubit a
        # complex multiply-add (TFIM: about 2.6 N Chebyshev terms of N + 1 each at this
        # field and step), 32 flops per gate
        N = case["N"]
        ops = case["steps"] * (2.6 * N) * (N + 1) * 4 if kind == "tfim" else \
            case["layers"] * (N - 1) * 32
        return {"bytes": 16 << N, "flops": int(ops * 2 ** N)}
    elem = 16 if case["dtype"] == C128 else 8
    if kind == "batch":
        sizes = _batch_sizes(case)
        return {"bytes": sum((elem << N) + 32 for N in sizes),
                "flops": sum((N + 4) << (2 * N) for N in sizes)}
    # one real value per Pauli string: N - 1 additions, product and reduction
    N = case["N"]
    shifts = case.get("x_count", 1 << N)
    out = 8 * shifts if kind == "shard" or case.get("partials") else 0
    if kind == "spectrum":
        out = 8 * case["nbins"]
    return {"bytes": (elem << N) + out + 32, "flops": shifts * (N + 4) << N}


# --- the same results in 64 bits, in plain torch ---------------------------

def _hadamard(n):
    h = torch.ones(1, 1, dtype=torch.float64, device="cuda")
    for _ in range(n):
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h


def _reduce(psi, N, x_count, fn):
    """fn(w, first shift), w = |W_x(z)|^2 (shifts x 2^N), over blocks of shifts."""
    D = 1 << N
    lo = N // 2
    hl, hh = _hadamard(lo), _hadamard(N - lo)
    k = torch.arange(D, device="cuda")
    p = psi.to(torch.complex128)
    step = max(1, min(x_count, (1 << 25) >> N))
    for x0 in range(0, x_count, step):
        xs = torch.arange(x0, min(x0 + step, x_count), device="cuda")
        f = p[k[None, :] ^ xs[:, None]].conj() * p[None, :]
        w = torch.zeros(len(xs), D, dtype=torch.float64, device="cuda")
        for part in (f.real, f.imag):
            t = part.reshape(-1, 1 << lo) @ hl
            t = t.reshape(len(xs), 1 << (N - lo), 1 << lo).transpose(1, 2).contiguous()
            t = t.reshape(-1, 1 << (N - lo)) @ hh
            w += t.reshape(len(xs), D) ** 2
        fn(w, x0)


def _pauli_sum(psi, alpha):
    N = psi.numel().bit_length() - 1
    sx = torch.zeros(1 << N, dtype=torch.float64, device="cuda")

    def add(w, x0):
        if alpha == 1.0:
            t = torch.where(w > 0, w * torch.log2(w.clamp_min(1e-300)), torch.zeros_like(w))
        else:
            t = w ** alpha
        sx[x0:x0 + len(w)] = t.sum(1)

    _reduce(psi, N, 1 << N, add)
    n = float((psi.to(torch.complex128).abs() ** 2).sum())
    S = float(sx.sum())
    if alpha == 1.0:
        m = math.log2(n * n) - S / (2.0 ** N * n * n)
    else:
        m = math.log2(S / (2.0 ** N * n ** (2 * alpha))) / (1.0 - alpha)
    return m, S, n, sx


def exact(case, seed):
    kind = case["kind"]
    if kind in ("tfim", "circuit"):
        return _exact_dynamics(case, seed)
    st = prepare(case, seed)
    if kind == "batch":
        rows = [_pauli_sum(p, 2.0)[:3] + (0.0,) for p in st["psi"]]
        return np.array(rows)
    psi, N = st["psi"], case["N"]
    shifts = case.get("x_count", 1 << N)
    if kind != "spectrum" and shifts << N > 1 << 35:
        return None
    if kind == "m2":
        m, S, n, sx = _pauli_sum(psi, 2.0)
        out = torch.tensor([m, S, n, 0.0], dtype=torch.float64)
        return (out, sx) if case["partials"] else (out,)
    if kind == "sre":
        return np.array(_pauli_sum(psi, case["alpha"])[:3])
    if kind == "spectrum":  # a count at a bin edge has no one value
        return {"counts": None, "n": float((psi.to(torch.complex128).abs() ** 2).sum())}
    sx = torch.zeros(shifts, dtype=torch.float64, device="cuda")

    def keep(w, x0):
        sx[x0:x0 + len(w)] = (w * w).sum(1)

    _reduce(psi, N, shifts, keep)
    return sx


def _exact_dynamics(case, seed):
    N = case["N"]
    st = prepare(case, seed)
    psi = torch.ones(1, dtype=torch.complex128, device="cuda")
    for t, p in zip(st["theta"], st["phi"]):  # qubit i is bit i
        one = torch.tensor([math.cos(t / 2), complex(math.cos(p), math.sin(p)) * math.sin(t / 2)],
                           dtype=torch.complex128, device="cuda")
        psi = (one[:, None] * psi[None, :]).reshape(-1)
    if case["kind"] == "circuit":
        for g, (q, _) in zip(st["gates"], st["pairs"]):
            u = torch.from_numpy(np.ascontiguousarray(g)).to("cuda")
            v = psi.reshape(-1, 4, 1 << int(q))
            psi = sum(u[:, j][None, :, None] * v[:, j][:, None, :]
                      for j in range(4)).reshape(-1)
        return psi
    J, hx, hz, dt = TFIM
    k = torch.arange(1 << N, device="cuda")
    z = [1.0 - 2.0 * ((k >> i) & 1).double() for i in range(N)]
    diag = -hz * sum(z) - J * sum(z[i] * z[i + 1] for i in range(N - 1))
    for _ in range(case["steps"]):
        sub = int(math.ceil((J * (N - 1) + (hx + hz) * N) * dt))  # |H dt| <= 1 each
        for _ in range(sub):
            term, acc = psi, psi.clone()
            for m in range(1, 22):  # Taylor series, 1 / 21! below 64 bits
                h = diag * term
                for i in range(N):
                    h = h - hx * term[k ^ (1 << i)]
                term = h * (-1j * dt / sub / m)
                acc += term
            psi = acc
    return psi
