"""The geometric graphs' block kernels at the edges of their rules: one cell or
2^D cells per block, 8 or 16 result words, the lane-per-vertex kernels beyond
the densest grid, radii from zero to the cell side (where every 16-bit distance
in the window matters), and blocks whose candidates exceed their words.  Byte
for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu

# points per cell on both sides of each rule's line
CASES = [(2, 6, a, f) for a in (1.0, 7.99, 8.0, 15.0, 31.9, 32.1) for f in (1.0, 0.6)]
CASES += [(3, 4, a, f) for a in (1.0, 4.99, 5.0, 9.99, 10.0, 21.9, 22.1) for f in (1.0, 0.7)]
CASES += [(2, 7, 3.0, 0.0), (2, 7, 12.0, 1e-3), (3, 4, 3.0, 0.0), (3, 4, 7.0, 1e-3)]


@pytest.mark.parametrize("d,L,a,f", CASES)
def test_blocks_equal_oracle(kgref, d, L, a, f):
    import torch
    kg = require_gpu()
    n = max(int(a * 2 ** (d * L)), 2 ** (d * L))
    r = f * 2.0 ** -L
    call, want_of = (kg.rgg2d, kgref.rgg2d) if d == 2 else (kg.rgg3d, kgref.rgg3d)
    points, edges = call(n, r, seed=31)
    torch.cuda.synchronize()
    want_points, want_edges = want_of(n, r, 31)
    assert np.array_equal(points.cpu().numpy().view(np.uint64), np.asarray(want_points).view(np.uint64).reshape(n, d))
    assert np.array_equal(to_np_u32(edges), want_edges)
