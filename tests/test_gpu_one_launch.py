"""Directed G(n,m) jobs of one launch, whose waves walk the chunk tree too: one
chunk, chunk counts around the 64 looked at together and around the rule's
limit, chunks of one row, several tiles per chunk, the last tile ragged, and as
many tiles as the rule takes.  Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,P", [
    (2, 1, 1), (2, 2, 2), (70, 500, 70), (130, 3000, 129), (5000, 60_000, 1), (5000, 60_000, 2), (5000, 60_000, 128),
    (5000, 60_000, 191), (5000, 60_000, 1023), (5000, 60_000, 1024), (5000, 60_000, 1025), (2**12, 2**16, 8),
    (2**16, 2**20, 64), (2**17 + 3, 2_200_000, 31), (3000, 8_000_000, 3)])
def test_one_launch_equals_oracle(kgref, n, m, P):
    import torch
    kg = require_gpu()
    want = kgref.generate(kgref.inst(n, m=m, directed=True, seed=12, chunks=P))
    for call in (kg.gnm, kg.gnm_static):
        got = call(n, m, True, 12, P)
        torch.cuda.synchronize()
        assert np.array_equal(to_np_u32(got), want), call.__name__
