"""CPU checks of the on-chip half transforms (k_half): every plan that the kernel
is compiled with, its LDS buffer of one real part, the maps from a shift's
elements to state indices, and shift 0's bit order.

The host-compiled maps and rounds are replayed in numpy: in FP64 against the
oracle's transform of single shifts, and in FP32 against the plain transform
in its own order of stages, bit for bit where the kernel relies on that (W_0; the
histogram's values)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import workloads as W
from test_plan import bfly, lane_bits, mapping, mf_reg_index, pad_np, round_math

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "half_probe.cpp")
M2, HIST, SPLIT = 0, 1, 2


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("half") / "half_probe.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so, SRC], check=True)
    lib = ctypes.CDLL(so)
    lib.probe_slot.restype = ctypes.c_uint
    return lib


class Half:
    def __init__(self, lib, prec, N, kind):
        out, zero = (ctypes.c_uint * 48)(), (ctypes.c_int * N)()
        rb, reals = ctypes.c_int(), ctypes.c_int()
        n = lib.probe_half(prec, N, kind, out, ctypes.byref(rb), ctypes.byref(reals), zero)
        assert n >= 1, (prec, N, kind)
        self.N, self.NT, self.rb, self.reals, self.zero = N, N - 1, rb.value, reals.value, list(zero)
        self.rounds = [tuple(out[6 * j:6 * j + 6]) for j in range(n)]

    def run(self, X):
        """The rounds on a tile of 2^NT values (leading axes: several tiles);
        the real and the imaginary parts pass the buffer one after the other."""
        E = [mapping(r, self.NT, self.rb) for r in self.rounds]
        V = round_math(X[..., E[0]], self.rounds[0])
        for j in range(1, len(self.rounds)):
            nxt = np.empty_like(V)
            for part in ("real", "imag"):
                lds = np.full(X.shape[:-1] + (self.reals,), np.nan, dtype=V.real.dtype)
                lds[..., pad_np(5, E[j - 1])] = getattr(V, part)
                getattr(nxt, part)[...] = lds[..., pad_np(5, E[j])]
            assert not np.isnan(nxt).any()
            V = round_math(nxt, self.rounds[j])
        out = np.empty_like(X)
        out[..., E[-1]] = V
        return out


def instances(lib):
    for prec in (0, 1):
        for kind in (M2, HIST, SPLIT):
            lo, hi = ctypes.c_int(), ctypes.c_int()
            if lib.probe_range(prec, kind, ctypes.byref(lo), ctypes.byref(hi)):
                continue
            for N in range(lo.value, hi.value + 1):
                yield prec, kind, N, Half(lib, prec, N, kind)


def k_map(lib, N, x, hist, last):
    k = np.empty(1 << (N - 1), np.uint32)
    hb = lib.probe_map(N, ctypes.c_uint(x), hist, last, ctypes.c_void_p(k.ctypes.data))
    return hb, k.astype(np.int64)


def shifts_of(N):
    """Shifts whose set bits lie in the top five bits, the low five, between
    them, and in several of these."""
    top, low, mid = 1 << (N - 1), 0b10110, 1 << 6
    return [1, 2, low, mid, mid | 3, top, top | (1 << (N - 5)), top >> 2, top | low, top | mid,
            (1 << N) - 1, (top >> 1) | mid | 1]


def test_ranges(probe):
    got = {}
    for prec, kind, N, _ in instances(probe):
        got.setdefault((prec, kind), []).append(N)
    assert got[0, M2] == list(range(10, 17)) and got[1, M2] == list(range(10, 16))
    assert got[0, HIST] == list(range(12, 15)) and got[1, HIST][-1] == 15
    assert got[0, SPLIT] == list(range(13, 17)) and (1, SPLIT) not in got


def test_plans(probe):
    """Every tile bit is a register, a lane or a wave bit of a round, gets one
    butterfly (or H_16 factor) in all, and a round's lanes hit distinct banks:
    32 lanes, 32 distinct slots modulo 32, in buffers of floats and doubles.  In
    the last round of N = 10 and 11 two lanes share one: the three or four
    register bits in the middle leave lane bits of too few residues modulo 5."""
    for prec, kind, N, h in instances(probe):
        case, seen = (prec, kind, N), 0
        threads = 1 << (h.NT - h.rb)
        assert 64 <= threads <= 1024, case
        assert h.reals * (4 if prec == 0 else 8) <= 160 * 1024 - 4096 - 512, case
        for rd in h.rounds:
            reg, bf, lane, wave, _, mf = rd
            assert reg | lane | wave == (1 << h.NT) - 1 and not (reg & lane | reg & wave | lane & wave)
            assert bin(reg).count("1") == h.rb and bin(lane).count("1") == 6, case
            assert sum(1 << b for b in lane_bits(rd)) == lane, case
            assert bf & ~reg == 0 and (bf | mf) & seen == 0, case
            assert (mf != 0) <= (kind == SPLIT), case
            if mf:
                assert mf_reg_index(rd) + 1 < h.rb and bin(mf & reg).count("1") == 2
                assert mf & lane == sum(1 << b for b in lane_bits(rd)[4:]), case
            seen |= bf | mf
        assert seen == (1 << h.NT) - 1, case
        if len(h.rounds) == 1:
            continue
        slots = pad_np(5, np.arange(1 << h.NT))
        assert slots[-1] + 1 == h.reals and np.all(np.diff(slots) > 0), case
        assert [probe.probe_slot(int(e)) for e in (0, 33, (1 << h.NT) - 1)] == \
            [slots[e] for e in (0, 33, (1 << h.NT) - 1)]
        for j, rd in enumerate(h.rounds):
            bank = (pad_np(5, mapping(rd, h.NT, h.rb)) % 32).reshape(threads // 32, 32, -1)
            ways = max(np.bincount(c, minlength=32).max()
                       for c in bank.transpose(0, 2, 1).reshape(-1, 32))
            two = N <= 11 and j == len(h.rounds) - 1
            assert ways == (2 if two else 1), (case, rd, ways)


@pytest.mark.parametrize("prec", [0, 1])
def test_maps_and_rounds_give_the_shift_transform(probe, oracle_mod, prec):
    """k covers the half space with bit hb of x clear; 2 Re A and 2i Im A of the
    replayed rounds are the oracle's W_x(z) at z = k(e) and k(e) + 2^hb."""
    for p, kind, N, h in instances(probe):
        if p != prec or N > 14:  # the larger ones differ in nothing but NT
            continue
        psi = W.haar(N, 5100 + N, np.complex128)
        for x in shifts_of(N):
            for last in ((0, 1) if kind == HIST and prec == 0 else (0,)):
                case = (prec, kind, N, x, last)
                hb, k = k_map(probe, N, x, int(kind == HIST), last)
                assert (x >> hb) & 1, case
                assert np.array_equal(np.sort(k), np.flatnonzero(~(np.arange(1 << N) >> hb) & 1))
                # disjoint parts of e stay disjoint (uniform and thread address parts)
                e = np.arange(1 << h.NT)
                reg = h.rounds[0][0]
                assert np.array_equal(k, k[e & reg] | k[e & ~reg]), case
                assert not np.any(k[e & reg] & k[e & ~reg]), case
                A = h.run(np.conj(psi[k ^ x]) * psi[k])
                ref = oracle_mod.shift_transform(psi, x)
                w0, w1 = ref[k], ref[k | (1 << hb)]
                sure = np.abs(w0.imag) < 1e-12  # W_x(z) is real or imaginary
                assert np.max(np.abs(np.where(sure, w0.real - 2 * A.real,
                                              w0.imag - 2 * A.imag))) < 1e-11, case
                assert np.max(np.abs(np.where(sure, w1.imag - 2 * A.imag,
                                              w1.real - 2 * A.real))) < 1e-11, case


def plain(lib, prec, N, f):
    """The plain transform in its own order of stages, in f's precision; the
    result at index z of the transform."""
    order = (ctypes.c_int * N)()
    lib.probe_plain_order(prec, N, order)
    assert sorted(order) == list(range(N))
    v = f.copy()
    for b in order:
        y = v.reshape(-1, 2, 1 << b)
        a, c = y[:, 0].copy(), y[:, 1].copy()
        y[:, 0], y[:, 1] = a + c, a - c
    return v


def test_shift_zero_keeps_the_plain_order(probe):
    """The two halves of |psi|^2 in the real and imaginary part and one stage
    across them: the plain transform's FP32 values, bit for bit."""
    for prec, kind, N, h in instances(probe):
        if prec or kind == SPLIT:
            continue
        assert sorted(h.zero) == list(range(N))
        rng = np.random.default_rng(N)
        f = rng.random(1 << N).astype(np.float32)
        e = np.arange(1 << h.NT)
        q = sum(((e >> b) & 1) << h.zero[b] for b in range(h.NT))
        last = 1 << h.zero[h.NT]
        X = np.empty(1 << h.NT, np.complex64)
        X.real, X.imag = f[q], f[q | last]
        A = h.run(X)
        ref = plain(probe, 0, N, f)
        # transform index of element e: the same bits
        assert np.array_equal(A.real + A.imag, ref[q]), (kind, N)
        assert np.array_equal(A.real - A.imag, ref[q | last]), (kind, N)


def test_histogram_values_keep_the_plain_bits(probe):
    """HB_LAST: 2 Re A and 2 Im A are the plain FP32 transform's values; the
    zero parts of those are exactly zero."""
    for prec, kind, N, h in instances(probe):
        if prec or kind != HIST:
            continue
        rng = np.random.default_rng(N)
        re, im = (rng.standard_normal(1 << N).astype(np.float32) for _ in range(2))
        idx = np.arange(1 << N)
        for x in shifts_of(N):
            f = np.empty(1 << N, np.complex64)
            f.real = re[idx ^ x] * re + im[idx ^ x] * im
            f.imag = re[idx ^ x] * im - im[idx ^ x] * re
            hb, k = k_map(probe, N, x, 1, 1)
            A = h.run(f[k])
            ref = plain(probe, 0, N, f)
            w0, w1 = ref[k], ref[k | (1 << hb)]
            real = w0.imag == 0
            assert np.array_equal(np.where(real, w0.real, w1.real), 2 * A.real), (N, x)
            assert np.array_equal(np.where(real, w1.imag, w0.imag), 2 * A.imag), (N, x)
            assert np.all(np.where(real, w1.real, w0.real) == 0), (N, x)


def test_rounds_of_the_largest_sizes(probe):
    """N = 15 and 16: the rounds are the Walsh-Hadamard transform of the tile."""
    for prec, kind, N, h in instances(probe):
        if N < 15:
            continue
        rng = np.random.default_rng(N + kind)
        X = rng.standard_normal(1 << h.NT) + 1j * rng.standard_normal(1 << h.NT)
        want = bfly(X[None, :], (1 << h.NT) - 1, (1 << h.NT) - 1)[0]
        assert np.max(np.abs(h.run(X) - want)) < 1e-10, (prec, kind, N)
