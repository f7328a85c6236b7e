"""Geometric graphs whose quadrant (octant) recursion takes three launches (more
than 24 binary levels): every vertex lies in its cell's range, and sampled cells'
counts and points equal the oracle's, which walks each cell's own root path."""
import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,r,L", [(2, 2**26 + 1, 1e-5, 13), (3, 2**27 + 77, 1e-4, 9)])
def test_three_launches(kgref, d, n, r, L):
    import torch
    kg = require_gpu()
    seed = 6
    level, path, cell_points = ((kgref.rgg_level, kgref.rgg_cell_count_path, kgref.rgg_cell_points) if d == 2 else
                                (kgref.rgg3_level, kgref.rgg3_cell_count_path, kgref.rgg3_cell_points))
    assert level(n, r) == L
    points, _ = (kg.rgg2d if d == 2 else kg.rgg3d)(n, r, seed=seed)
    z = torch.zeros(n, dtype=torch.int64, device="cuda")
    for a in range(d):
        c = (points[:, a] * 2.0**L).to(torch.int64)
        for b in range(L):
            z |= ((c >> b) & 1) << (d * b + a)
    assert bool((z[1:] >= z[:-1]).all())
    cells = torch.bincount(z, minlength=2 ** (d * L))
    assert int(cells.sum()) == n and cells.numel() == 2 ** (d * L)
    first = torch.cumsum(cells, 0) - cells
    rng = np.random.default_rng(8)
    for q in [0, 1, 2 ** (d * L) - 1] + [int(x) for x in rng.integers(0, 2 ** (d * L), 300)]:
        k, at = int(cells[q]), int(first[q])
        assert k == path(n, r, seed, q), q
        got = points[at:at + k].cpu().numpy()
        want = np.asarray(cell_points(n, r, seed, q, k))
        assert np.array_equal(got.view(np.uint64).reshape(-1), want.view(np.uint64).reshape(-1)), q
