"""Deep tile trees: a batch whose planner starts below the chunks' roots, and
units over several rounds of lanes, against the same graphs one at a time (whose
planner walks from the root), and one of them against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [0, 1])
def test_batch_equals_single_graphs(kgref, waves):
    import torch
    kg = require_gpu()
    # graphs of about 17,000 tiles: single chunks of odd sizes, a few of several
    # chunks (as deep as the rule's line, below it, and of one tile)
    shapes = [(4_300_037 + 999 * i, 10_500_000 + 1001 * i, i % 2 == 0, 1) for i in range(13)]
    shapes += [(2_000_003, 8_000_000, True, 31), (2_000_003, 8_000_000, False, 33), (3000, 70_000, True, 70)]
    insts = [kg.Instance(n, kg.GNM, d, m, 0.0, 100 + i, P) for i, (n, m, d, P) in enumerate(shapes)]
    try:
        kg.set_option(kg._lib.KG_OPT_PLAN_WAVES, waves)
        edges, offsets = kg.batch(insts)
        torch.cuda.synchronize()
    finally:
        kg.set_option(kg._lib.KG_OPT_PLAN_WAVES, 0)
    at = offsets.cpu().numpy().astype(np.int64)
    for i, (n, m, d, P) in enumerate(shapes):
        one = kg.gnm(n, m, d, 100 + i, P)
        torch.cuda.synchronize()
        assert at[i + 1] - at[i] == m
        assert torch.equal(edges[at[i]:at[i + 1]].view(torch.int32), one.view(torch.int32)), i
    n, m, d, P = shapes[1]
    want = kgref.generate(kgref.inst(n, m=m, directed=d, seed=101, chunks=P))
    assert np.array_equal(to_np_u32(edges[at[1]:at[2]]), want)
