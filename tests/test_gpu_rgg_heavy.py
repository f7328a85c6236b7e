"""Geometric graphs with blocks whose window holds more candidates than the
block's result words have bits: those blocks are tested in binary64 in both edge
passes.  The seeds give at least one such block, which the oracle's cell
counts prove before the comparison, byte for byte, with the oracle's edges."""
import itertools

import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

# dimension, level, points per cell, block level, result words per vertex, seed
CASES = [(3, 5, 4.99, 1, 8, 1), (3, 6, 9.99, 0, 8, 1), (3, 5, 21.9, 0, 16, 2), (2, 8, 31.99, 0, 8, 18)]


def spread(x, d):
    """The bits of x, d places apart."""
    x = np.asarray(x, dtype=np.int64)
    return sum(((x >> b) & 1) << (d * b) for b in range(16))


def most_candidates(counts, d, L, B):
    """The largest number of points, over the blocks of 2^B cells a side, in the
    cells of the block's window (one cell around it) from its first cell on."""
    g, b = 1 << L, 1 << B
    z = sum(spread(c, d) << a for a, c in enumerate(np.meshgrid(*[np.arange(g)] * d, indexing="ij")))
    inner = (slice(1, -1),) * d
    index, points = np.full([g + 2] * d, -1, dtype=np.int64), np.zeros([g + 2] * d, dtype=np.int64)
    index[inner], points[inner] = z, np.asarray(counts).astype(np.int64)[z]
    first = z[(slice(None, None, b),) * d]
    total = np.zeros_like(first)
    for off in itertools.product(range(b + 2), repeat=d):
        at = tuple(slice(o, o + g - b + 1, b) for o in off)
        total += np.where(index[at] >= first, points[at], 0)
    return int(total.max())


@pytest.mark.gpu
@pytest.mark.parametrize("d,L,a,B,words,seed", CASES)
def test_heavy_blocks_equal_oracle(kgref, d, L, a, B, words, seed):
    import torch
    kg = require_gpu()
    n, r = int(a * 2 ** (d * L)), 0.51 * 2.0 ** -L
    cells, graph = (kgref.rgg_cells, kgref.rgg2d) if d == 2 else (kgref.rgg3_cells, kgref.rgg3d)
    assert most_candidates(cells(n, r, seed), d, L, B) > 32 * words
    points, edges = (kg.rgg2d if d == 2 else kg.rgg3d)(n, r, seed=seed)
    torch.cuda.synchronize()
    want_points, want_edges = graph(n, r, seed)
    assert np.array_equal(points.cpu().numpy().view(np.uint64), np.asarray(want_points).view(np.uint64).reshape(n, d))
    assert np.array_equal(to_np_u32(edges), want_edges)
