"""Row and column of a slot where the row width is no power of two: widths on
both sides of powers of two (both forms of the reciprocal multiplier), the
smallest and the largest, directed (rows of n - 1 slots) and undirected
(rectangles as wide as a section).  Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu

WIDTHS = [3, 5, 6, 7, 9, 11, 641, 2**12 - 1, 2**12 + 1, 2**16 - 1, 2**16 + 1, 99991, 3 * 2**18, 2**20 - 1, 2**20 + 1,
          2**22 - 1, 2**22 + 1]


@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("directed", [True, False])
def test_rows_equal_oracle(kgref, width, directed):
    import torch
    kg = require_gpu()
    chunks = 3
    n = width + 1 if directed else chunks * width
    slots = n * (n - 1) // (1 if directed else 2)
    # tiles of at most 2^31 slots, so that 32-bit positions take the multiplier
    m = min(slots * 2 // 5, max(150000, slots * 600 // 2**31))
    got = kg.gnm(n, m, directed, 5, chunks)
    torch.cuda.synchronize()
    want = kgref.generate(kgref.inst(n, m, directed=directed, seed=5, chunks=chunks))
    assert np.array_equal(to_np_u32(got), want)
