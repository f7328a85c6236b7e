"""Jobs with tiles of 2^32 slots on the persistent grid: tiles of one key to more
than three rounds of 256 draws hold, with the keys per lane and the rounds of
the base case's copies changing in between, ragged last tiles of 2^31 slots and
more (rejections) and of a few, a batch that mixes them with smaller tiles, and
tiles whose draws hold a repeat.  Byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keys", [0.5, 3, 60, 250, 256, 262, 500, 512, 524, 735, 752, 768, 780, 1024, 1110])
def test_whole_tiles_equal_oracle(kgref, keys):
    import torch
    kg = require_gpu()
    n, tiles = 3200003, 2385                     # 3200003 * 3200002 / 2^32 = 2384.2
    m = int(keys * 2384)
    I = kgref.inst(n, m=m, directed=True, seed=3, chunks=1)
    assert kgref.tile_exponent(I) == 32
    got = kg.gnm(n, m, directed=True, seed=3, chunks=1)
    torch.cuda.synchronize()
    assert np.array_equal(to_np_u32(got), kgref.generate(I))


@pytest.mark.parametrize("n,m,directed,chunks", [
    (2**17 + 1, 2**20, True, 2900), (2**23 + 5, 3 * 10**6, False, 90), (2**16, 10**5, True, 2**16),
    (2**23, 4 * 10**6, False, 64), (5 * 10**6, 2 * 10**6, True, 3001)])
def test_ragged_tiles_equal_oracle(kgref, n, m, directed, chunks):
    import torch
    kg = require_gpu()
    N = n * (n - 1) // (1 if directed else 2)
    p = min(m / N, 2.5e-7)
    I = kgref.inst(n, p=p, directed=directed, seed=4, chunks=chunks)
    assert kgref.tile_exponent(I) == 32
    got = kg.gnp(n, p, directed=directed, seed=4, chunks=chunks)
    torch.cuda.synchronize()
    assert np.array_equal(to_np_u32(got), kgref.generate(I))


def test_mixed_batch_equals_oracle(kgref):
    import torch
    kg = require_gpu()
    specs = [(3200003, 2**20, True, 7), (2**14, 2**20, False, 3), (2**22, 2**19, False, 11), (5000, 2**18, True, 1)]
    arena, offs = kg.batch([kg.Instance(n, kg.GNM, d, m, 0.0, 9 + i, P) for i, (n, m, d, P) in enumerate(specs)])
    torch.cuda.synchronize()
    O = to_np_u64(offs).astype(np.int64)
    for i, (n, m, d, P) in enumerate(specs):
        want = kgref.generate(kgref.inst(n, m=m, directed=d, seed=9 + i, chunks=P))
        assert np.array_equal(to_np_u32(arena[O[i]:O[i + 1]]), want), i


@pytest.mark.parametrize("keys,seed", [(500, 1), (1000, 1)])
def test_repeats_equal_oracle(kgref, keys, seed):
    """The oracle's tile counts and streams prove that a tile draws a value twice."""
    import torch
    kg = require_gpu()
    n, tiles = 12 * 10**6, 33527                 # n (n - 1) / 2^32
    m = keys * tiles
    I = kgref.inst(n, m=m, directed=True, seed=seed, chunks=1)
    assert kgref.tile_exponent(I) == 32
    K = kgref.tile_counts(I, 0, m)[:tiles].astype(np.int64)
    most, repeats = 4 * ((int(K.max()) + 3) // 4), 0
    for t0 in range(0, tiles, 4096):
        k = K[t0:t0 + 4096]
        rec = np.zeros((len(k), most // 4, 6), dtype=np.uint32)
        rec[:, :, 1] = np.arange(most // 4)
        rec[:, :, 2] = np.arange(t0, t0 + len(k))[:, None]
        rec[:, :, 3] = kgref.TAG_TLEAF
        rec[:, :, 4] = seed
        x = kgref.eval_many(1, rec.reshape(-1, 6), np.uint32, 4).reshape(len(k), most).astype(np.int64)
        x[np.arange(most)[None, :] >= k[:, None]] = -1
        x.sort(axis=1)
        repeats += int(((x[:, 1:] == x[:, :-1]) & (x[:, 1:] >= 0)).sum())
    assert repeats > 0
    got = kg.gnm(n, m, directed=True, seed=seed, chunks=1)
    torch.cuda.synchronize()
    assert np.array_equal(to_np_u32(got), kgref.generate(I))
