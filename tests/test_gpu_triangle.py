"""Triangle chunks (Sec. 4.2) in one section: tiles of 2^31 slots whose rows
run from 2^24 slots down to one (32-bit decode up to its limits), one tile
holding a whole small triangle, and tiles of 2^32 slots (general decode)."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(2**24 + 5, 40_000_000), (2, 1), (40, 300), (1201, 700), (70000, 3_000_000),
                                 (2**27 + 3, 1_000_000)])
def test_one_section(kgref, n, m):
    import torch
    kg = require_gpu()
    got = kg.gnm(n, m, directed=False, seed=9, chunks=1)
    torch.cuda.synchronize()
    want = kgref.generate(kgref.inst(n, m=m, directed=False, seed=9, chunks=1))
    assert np.array_equal(to_np_u32(got), want)
