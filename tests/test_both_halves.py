"""CPU checks of the full slab that row pairs are compared with: its rows are
transformed in two halves (row bit j clear, set) and combined last
(sre2_both.h).  Its terms have to depend on both halves, or the comparison
says nothing; and on a shift's own slab they have to be the half slab's
16 (Re^4 + Im^4), bit for bit.

The first is compared in FP64 with |v + u|^4 + |v - u|^4; the terms square
FP32 values, so they carry 4 roundings of 6e-8 each: 1e-6."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "both_probe.cpp")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("both") / "both_probe.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so, SRC], check=True)
    return ctypes.CDLL(so)


def terms(lib, v, u, odd):
    v, u = (np.ascontiguousarray(a, np.complex64).reshape(-1) for a in (v, u))
    odd = np.ascontiguousarray(odd, np.uint32).reshape(-1)
    out = np.empty(v.size)
    p = ctypes.c_void_p
    lib.probe_terms(p(v.ctypes.data), p(u.ctypes.data), p(odd.ctypes.data), v.size,
                    p(out.ctypes.data))
    return out


def wht(a, axis):
    """Unnormalised transform along one axis, in the array's own precision."""
    a = np.moveaxis(a, axis, -1).copy()
    n = a.shape[-1]
    h = 1
    while h < n:
        b = a.reshape(a.shape[:-1] + (n // (2 * h), 2, h))
        p, q = b[..., 0, :].copy(), b[..., 1, :].copy()
        b[..., 0, :], b[..., 1, :] = p + q, p - q
        h *= 2
    return np.moveaxis(a, -1, axis)


@pytest.mark.parametrize("u_of", ["independent", "zero", "same", "opposite"])
def test_terms_count_both_halves(probe, u_of):
    rng = np.random.default_rng(7)
    v, w = ((rng.standard_normal(256) + 1j * rng.standard_normal(256)).astype(np.complex64)
            for _ in range(2))
    u = {"independent": w, "zero": 0 * v, "same": v, "opposite": -v}[u_of]
    v8, u8 = v.astype(np.complex128), u.astype(np.complex128)
    want = np.abs(v8 + u8) ** 4 + np.abs(v8 - u8) ** 4
    for odd in (0, 1):
        got = terms(probe, v, u, np.full(256, odd))
        assert np.max(np.abs(got - want) / want) <= 1e-6
    # what half the slab alone would say
    assert np.max(np.abs(16 * (v8.real ** 4 + v8.imag ** 4) - want) / want) > 1e-2


@pytest.mark.parametrize("L,HB,CB", [(4, 4, 2), (5, 2, 3), (3, 5, 0)])
def test_slab_halves_agree_bitwise_with_the_half_slab(probe, L, HB, CB):
    """Slabs of 2^HB rows of 2^L values: the parity of the stored index picks
    the real value, and the terms are the half slab's in every bit."""
    N, T = L + HB, 1 << CB
    rng = np.random.default_rng(N)
    psi = (rng.standard_normal(1 << N) + 1j * rng.standard_normal(1 << N)).astype(np.complex64)
    re, im = psi.real, psi.imag
    k = np.arange(1 << N)
    for x in (1 << L, (1 << L) + 5, (3 << L) + 2, (1 << N) - 1, (1 << (N - 1)) + 6):
        xh, xl = x >> L, x & ((1 << L) - 1)
        j = xh.bit_length() - 1
        f = np.empty((1 << HB, 1 << L), np.complex64)
        f.real = (re[k ^ x] * re + im[k ^ x] * im).reshape(f.shape)
        f.imag = (re[k ^ x] * im - im[k ^ x] * re).reshape(f.shape)
        rows = wht(f, 1)
        r = np.arange(1 << HB)
        v, u = (wht(rows[((r >> j) & 1) == b], 0) for b in (0, 1))
        z = np.arange(1 << (HB - 1))[:, None], np.arange(1 << L)[None, :]
        e = (z[0] << CB) | (z[1] & (T - 1))  # element of the column tile z1 >> CB
        xt = probe.probe_mask(xh, xl, j, CB)
        par = np.vectorize(lambda a: probe.probe_parity(int(a)))
        odd = par(e & xt) ^ par((z[1] & ~(T - 1)) & xl)
        s = np.where(odd, -1, 1)
        assert np.array_equal(u.real, s * v.real) and np.array_equal(u.imag, -s * v.imag)
        a, b = (v.real * v.real).astype(np.float64), (v.imag * v.imag).astype(np.float64)
        # 16 fma(a, a, b b): a and b have 24 bits, so their products and the
        # rounded sum of them are what FP64 gives
        want = 16.0 * (a * a + b * b)
        assert np.array_equal(terms(probe, v, u, odd), want.reshape(-1))
