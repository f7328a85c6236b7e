"""Plane geometric graphs of about one to three points per cell, on both sides of
the lines below which a lane per vertex takes the edges instead of a block of
cells (2.1 points, 1.5 for a radius under an eighth of a cell; 4^9 cells and
more).  Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 8, 9])
@pytest.mark.parametrize("a", [1.0, 1.49, 1.51, 2.09, 2.11, 3.0])
@pytest.mark.parametrize("f", [1.0, 0.5, 0.126, 0.124, 1e-3, 0.0])
def test_few_points_equal_oracle(kgref, L, a, f):
    import torch
    kg = require_gpu()
    n, r = max(int(a * 4**L), 4**L), f * 2.0**-L
    assert kgref.rgg_level(n, r) == L
    points, edges = kg.rgg2d(n, r, seed=41)
    torch.cuda.synchronize()
    want_points, want_edges = kgref.rgg2d(n, r, 41)
    assert np.array_equal(points.cpu().numpy().view(np.uint64), np.asarray(want_points).view(np.uint64).reshape(n, 2))
    assert np.array_equal(to_np_u32(edges), want_edges)
