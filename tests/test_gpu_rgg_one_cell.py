"""Geometric graphs whose grid is one cell: radii from just above a cell side to
beyond the diagonal, where every point's circle covers its window's corner, at
most as many points as the block kernels take and one more.  Byte for byte
against the oracle, into a buffer that the edges fill exactly."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("r", [0.9, 1.2, 1.4142, 1.42, 1.5, 2.0, 3.0, 5.0, 1e6, float("inf")])
def test_one_cell_equals_oracle(kgref, d, r):
    import torch
    kg = require_gpu()
    call, want_of = (kg.rgg2d, kgref.rgg2d) if d == 2 else (kg.rgg3d, kgref.rgg3d)
    for n in (1, 2, 3, 5, 10, 17, 20, 22, 23, 31, 32, 33):
        for seed in (1, 2, 3, 4):
            want_points, want_edges = want_of(n, r, seed)
            out = torch.full((len(want_edges), 2), 7, dtype=torch.int32, device="cuda").view(torch.uint32)
            points, edges, total = call(n, r, seed=seed, out=out)
            torch.cuda.synchronize()
            assert int(to_np_u64(total)[0]) == len(want_edges), (n, seed)
            assert np.array_equal(to_np_u32(edges), want_edges), (n, seed)
            assert np.array_equal(points.cpu().numpy().view(np.uint64),
                                  np.asarray(want_points).view(np.uint64).reshape(n, d)), (n, seed)
