"""Launch rules of small jobs: offsets from the count kernel's one workgroup
(up to 64 chunks), from one workgroup's scan (up to 4,096) or from the
three-phase scan; a wave per tile that walks the tile tree itself (few tiles per
compute unit) or the planner and the queue; with the general base case forced
too.  Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf_cap", [0, 128])
@pytest.mark.parametrize("n,m,directed,P", [
    (3000, 70_000, True, 63), (3000, 70_000, True, 64), (3000, 70_000, True, 65), (3000, 70_000, False, 10),
    (3000, 70_000, False, 11), (20000, 300_000, True, 4096), (20000, 300_000, True, 4097), (20000, 300_000, False, 90),
    (20000, 300_000, False, 91), (2**17 + 3, 2_200_000, True, 1), (2**17 + 3, 2_400_000, True, 1),
    (2**17 + 3, 2_200_000, False, 9), (2**17 + 3, 2_500_000, False, 9), (1500, 2_000_000, True, 5), (40, 900, False, 1)])
def test_small_jobs_equal_oracle(kgref, n, m, directed, P, leaf_cap):
    import torch
    kg = require_gpu()
    m = min(m, n * (n - 1) // (1 if directed else 2))
    want = kgref.generate(kgref.inst(n, m=m, directed=directed, seed=6, chunks=P))
    try:
        kg.set_option(kg._lib.KG_OPT_LEAF_CAP, leaf_cap)
        got = kg.gnm(n, m, directed=directed, seed=6, chunks=P)
        torch.cuda.synchronize()
    finally:
        kg.set_option(kg._lib.KG_OPT_LEAF_CAP, 0)
    assert np.array_equal(to_np_u32(got), want)
