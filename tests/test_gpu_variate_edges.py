"""The variates' binary32 acceptance decision, the waiting times at p = 1/2
and the sections' divisions, where they change path: counts around the smallest
arguments the decision takes (y = 16), deviations around |t| = 0.2 and far
from the mode, means around 16, and sections at the largest sizes.  Bit for bit
against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32

pytestmark = pytest.mark.gpu
COUNT = 200000


@pytest.fixture(scope="module")
def kg():
    return require_gpu()


def _records(law, rng, n):
    seeds = [rng.integers(0, 2**63, n).astype(np.uint64), rng.integers(0, 2**63, n).astype(np.uint64),
             rng.integers(1, 7, n).astype(np.uint64)]
    if law.startswith("bin"):
        if law == "bin_half_small":            # both sides of N p = 16
            N, p = rng.integers(1, 130, n), np.full(n, 0.5)
        elif law == "bin_half_large":
            N, p = np.exp(rng.uniform(4, 30, n)).astype(np.int64), np.full(n, 0.5)
        else:                                  # means 16 .. 300 of every p
            N = np.exp(rng.uniform(4, 30, n)).astype(np.int64)
            p = np.minimum(rng.uniform(15, 300, n) / N, 0.5 - 1e-9 * rng.random(n))
        return 6, np.stack([N.astype(np.uint64), p.view(np.uint64), np.zeros(n, np.uint64)] + seeds, axis=1)
    if law == "hyp_tile":                      # leaves of the tile tree
        N, k = np.full(n, 2**23), rng.integers(1000, 2300, n)
        K = np.full(n, 2**22)
    elif law == "hyp_small":                   # some count of the law near 16
        k = rng.integers(17, 200, n)
        N = np.exp(rng.uniform(5.5, 40, n)).astype(np.int64)
        N = np.maximum(N, 2 * k + 2)
        K = np.clip(N * rng.uniform(10, 40, n) / k, 1, N - 1).astype(np.int64)
    else:                                      # large counts, even and uneven
        N = np.exp(rng.uniform(30, 43, n)).astype(np.int64)
        K = (N * rng.uniform(1e-3, 0.999, n)).astype(np.int64)
        k = np.exp(rng.uniform(12, 28, n)).astype(np.int64)
    return 5, np.stack([N.astype(np.uint64), K.astype(np.uint64), k.astype(np.uint64)] + seeds, axis=1)


@pytest.mark.parametrize("law", ["hyp_tile", "hyp_small", "hyp_large", "bin_half_small", "bin_half_large", "bin_mean"])
def test_variates_equal_oracle(kg, kgref, law):
    import torch
    fn, rec = _records(law, np.random.default_rng(71), COUNT)
    rec = np.ascontiguousarray(rec)
    d = torch.from_numpy(rec.view(np.int64)).cuda()
    got = kg.eval_device(fn, d, COUNT, torch.int64, 1).cpu().numpy().view(np.uint64)
    want = kgref.eval_many(fn, rec, np.uint64, 1)
    bad = np.nonzero(got[:, 0] != want[:, 0])[0]
    assert len(bad) == 0, (law, rec[bad[:5]])


@pytest.mark.parametrize("n,P,rank", [(2**32 - 5, 2**15, 12345), (2**32, 2**15 - 1, 2**15 - 2), (2**32, 1000, 999)])
def test_view_of_the_largest_sections(kg, kgref, n, P, rank):
    import torch
    m = 50_000_000
    got = kg.pe_view(n, rank, P, directed=False, m=m, seed=3)
    torch.cuda.synchronize()
    want = kgref.pe_view(kgref.inst(n, m=m, directed=False, seed=3, chunks=P), rank)
    assert np.array_equal(to_np_u32(got), want)
