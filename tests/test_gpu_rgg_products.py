"""Three-dimensional graphs whose tests are formed by the matrix units, on both
sides of the lines between one cell and eight cells per block, and at radii
where squares near the threshold are common (the same points for every radius,
so many distances fall into the margin taken for the products' rounding).  Byte
for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a", [4.5, 5.5, 7.49, 7.51])
@pytest.mark.parametrize("f", [1.0, 0.93, 0.7, 0.51, 0.2, 0.02])
def test_products_equal_oracle(kgref, a, f):
    import torch
    kg = require_gpu()
    L = 4
    n, r = int(a * 2 ** (3 * L)), f * 2.0 ** -L
    points, edges = kg.rgg3d(n, r, seed=77)
    torch.cuda.synchronize()
    want_points, want_edges = kgref.rgg3d(n, r, 77)
    assert np.array_equal(points.cpu().numpy().view(np.uint64), np.asarray(want_points).view(np.uint64).reshape(n, 3))
    assert np.array_equal(to_np_u32(edges), want_edges)


@pytest.mark.parametrize("a", [9.9, 10.1])
@pytest.mark.parametrize("f", [1.0, 0.6])
def test_plane_line_equals_oracle(kgref, a, f):
    """Two dimensions, on both sides of the line between one cell and four."""
    import torch
    kg = require_gpu()
    n, r = int(a * 2**14), f * 2.0**-7
    points, edges = kg.rgg2d(n, r, seed=78)
    torch.cuda.synchronize()
    want_points, want_edges = kgref.rgg2d(n, r, 78)
    assert np.array_equal(points.cpu().numpy().view(np.uint64), np.asarray(want_points).view(np.uint64).reshape(n, 2))
    assert np.array_equal(to_np_u32(edges), want_edges)
