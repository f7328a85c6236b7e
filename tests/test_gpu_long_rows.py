"""Directed views of more than 2^31 vertices, whose rows' remainders need all 32
bits, through the register base case (a wave per tile, and the persistent grid)
and the general one, which decodes slots by another routine.  Against the
oracle byte for byte."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu

# n, m, p, chunks, rank, tile exponent
NARROW = [(2**31 + 2, 7 * 10**12, None, 2**24, 5, 29), (3 * 10**9, 2 * 10**13, None, 2**24, 2**23, 28),
          (3 * 10**9, 2 * 10**13, None, 2**21, 77, 28), (3700000001, 0, 1.5e-6, 2**20, 2**19, 29)]


def check(kgref, n, m, p, P, rank, s):
    import torch
    kg = require_gpu()
    I = kgref.inst(n, m=m, p=p or 0.0, directed=True, seed=11, chunks=P)
    assert kgref.tile_exponent(I) == s
    want = kgref.pe_view(I, rank)
    for cap in (0, 128):
        kg.set_option(kg._lib.KG_OPT_LEAF_CAP, cap)
        try:
            got = kg.pe_view(n, rank, P, directed=True, m=m, p=p, seed=11)
            torch.cuda.synchronize()
        finally:
            kg.set_option(kg._lib.KG_OPT_LEAF_CAP, 0)
        assert np.array_equal(to_np_u32(got), want), cap


@pytest.mark.parametrize("n,m,p,P,rank,s", NARROW)
def test_long_rows_equal_oracle(kgref, n, m, p, P, rank, s):
    assert 2**31 < n - 1 <= 2**32 - 2**s
    check(kgref, n, m, p, P, rank, s)


# rows of more than 2^32 - 2^s slots: a tile that starts near a row's end has
# slots past 2^32 counted from that row's start, and the next tile starts in the
# row after
WIDE = [(4 * 10**9, 6 * 10**12, None, 6 * 10**6, 1234567, 31),
        (2**32 - 5, 2**43, None, 2**22, 77, 31), (2**32 - 5, 2**43, None, 2**20, 77, 31),
        (2**32, 2**44, None, 2**22, 2**22 - 1, 30), (3900000007, 2 * 10**13, None, 2**23, 3, 29),
        (2**32 - 1, 0, 2.7e-7, 2**20, 2**19, 31)]


@pytest.mark.parametrize("n,m,p,P,rank,s", WIDE)
def test_wide_rows_equal_oracle(kgref, n, m, p, P, rank, s):
    assert n - 1 > 2**32 - 2**s and s < 32
    check(kgref, n, m, p, P, rank, s)
