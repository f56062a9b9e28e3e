"""Geometry and workspace queries at the sizes that M2 evaluates on chip above the
fused kernel's: FP32 N = 15, 16, FP64 N = 14, 15 (host-only, no GPU needed).

Only the FP32 spectrum, SPLIT_BF16 and shift 0 of SPLIT_F16 take slabs there."""
import pytest

import paper_2512_24685_amd as sre2

ONCHIP = [("fp32", 15), ("fp32", 16), ("fp32h", 15), ("fp32h", 16), ("fp64", 14), ("fp64", 15),
          ("fp64h", 14), ("fp64h", 15)]


@pytest.fixture(scope="module")
def ctx():
    c = sre2.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("form,N", ONCHIP)
def test_no_slab_in_the_workspace(ctx, form, N):
    c64 = not form.startswith("fp64")
    got = sre2.lib().sre2_workspace_bytes(N, sre2.C64 if c64 else sre2.C128, sre2.FORMS[form])
    # S_x and the reduction buffers (below 64 KiB)
    assert 8 << N <= got <= (8 << N) + (64 << 10)
    assert ctx.chunking(N, form) == (0, 1)


@pytest.mark.parametrize("N", [15, 16])
def test_split_forms(ctx, N):
    L = sre2.lib()
    f16 = L.sre2_workspace_bytes(N, sre2.C64, sre2.FORMS["split16"])
    slab = 8 << N  # one shift
    assert (8 << N) + slab <= f16 <= (8 << N) + slab + (64 << 10)
    assert ctx.chunking(N, "split16") == (0, 1)
    cs, _ = ctx.chunking(N, "splitbf16")  # two passes: half slabs of 2^L shifts
    assert cs == 1 << sre2.row_bits(N, "splitbf16")
    bf16 = L.sre2_workspace_bytes(N, sre2.C64, sre2.FORMS["splitbf16"])
    assert bf16 >= cs * (4 << N)


def test_where_slabs_begin(ctx):
    for form in ("fp64", "fp64h"):
        for N in (14, 15):
            assert sre2.row_bits(N, form) == 0
            assert sre2.half_slab_first_shift(N, form) == 1 << N
        assert sre2.row_bits(16, form) == 11
        assert sre2.half_slab_first_shift(16, form) == 1 << 11
        assert ctx.chunking(16, form)[0] > 0
    for form in ("fp32", "fp32h", "split16"):
        assert ctx.chunking(17, form)[0] == 1 << 12
        # the spectrum's slabs, shift 0's
        assert sre2.row_bits(15, form) == 12 and sre2.row_bits(14, form) == 0
