"""The skip sampler's quick logarithm and its two position sums, where they
change path: tiles of 2^30, 2^31 (32-bit sums) and 2^32 slots (64-bit), gaps
near whole numbers (p around 1/2, where log U / L is small, and p so small
that the full logarithm decides every gap), with and without stored rows.
Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kgs():
    return require_gpu()


# 1024 / 2^31 = 4.77e-7 and 1024 / 2^30 = 9.54e-7: on either side of each
@pytest.mark.parametrize("n,p,directed", [
    (2**20, 4.7e-7, True), (2**20, 4.8e-7, True), (2**20, 9.6e-7, False), (2**20, 1e-10, True),
    (2**24, 1e-13, True), (2**24, 2e-14, False), (3000, 0.499999, True), (3000, 0.500001, False),
    (3000, 0.999999, True), (3000, 1.0 - 1e-12, True), (4000, 0.25, False)])
def test_gaps_equal_oracle(kgs, kgref, n, p, directed):
    import torch
    want = kgref.skip_generate(kgref.inst(n, p=p, directed=directed, seed=21, chunks=3, model=kgref.GNP))
    inst = kgs.Instance(n, kgs.GNP, directed, 0, p, 21, 3)
    small = torch.empty(kgs.workspace_bytes([inst]), dtype=torch.uint8, device="cuda")
    for what, ws in (("rows", None), ("regenerated", small)):
        got = kgs.gnp_skip(n, p, directed, 21, 3, workspace=ws)
        torch.cuda.synchronize()
        assert got.shape[0] == len(want), what
        assert np.array_equal(to_np_u32(got), want), what
