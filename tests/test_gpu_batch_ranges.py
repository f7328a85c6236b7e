"""Batches whose tiles are shared out in fixed ranges: fewer tiles than
workgroups, all tiles fixed, three quarters of them, and ranges taken from the
counter only; dense graphs (several times the cost per tile) beside sparse ones.
Byte for byte the same graphs one at a time, the first against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,edges", [(3, 400_000), (5, 5_000_000), (9, 8_000_003), (23, 20_000_003), (30, 24_000_000)])
def test_batch_equals_single_graphs(kgref, count, edges):
    import torch
    kg = require_gpu()
    shapes = []
    for i in range(count):
        d = i % 3 != 0
        n = int((edges * (4 if d else 8)) ** 0.5) if i % 4 == 1 else edges // 7 + i    # a quarter of the slots, or sparse
        shapes.append((n, edges + i if i else 300_000, d, 1 + 7 * (i % 5)))
    insts = [kg.Instance(n, kg.GNM, d, m, 0.0, 40 + i, P) for i, (n, m, d, P) in enumerate(shapes)]
    arena, offsets = kg.batch(insts)
    torch.cuda.synchronize()
    at = offsets.cpu().numpy().astype(np.int64)
    for i, (n, m, d, P) in enumerate(shapes):
        one = kg.gnm(n, m, d, 40 + i, P)
        torch.cuda.synchronize()
        assert at[i + 1] - at[i] == m
        assert torch.equal(arena[at[i]:at[i + 1]].view(torch.int32), one.view(torch.int32)), i
    n, m, d, P = shapes[0]
    want = kgref.generate(kgref.inst(n, m=m, directed=d, seed=40, chunks=P))
    assert np.array_equal(to_np_u32(arena[:at[1]]), want)
