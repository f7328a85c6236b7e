"""The skip sampler's count pass by a lane per tile (many tiles of few events) and
by a wave per tile, on both sides of the lines between them: tiles of no
event, of a few, of some hundred; whole tiles and the small ones of many chunks;
failures counted instead (p > 1/2); p = 0 and 1.  Totals of a call without
edges and the regenerated edges, against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32, to_np_u64

pytestmark = pytest.mark.gpu

# tiles: 2^8, 2^12, 2^14 of 2^32 slots, many chunks' part tiles, tiles of 1024 slots
CASES = [(2**20, e / 2.0**32, True, 1) for e in (0.01, 0.12, 0.13, 3.0)]
CASES += [(2**22, e / 2.0**32, True, 5) for e in (0.5, 1.9, 2.1, 40.0)]
CASES += [(2**23 + 5, e / 2.0**32, False, 3) for e in (3.9, 4.1)]
CASES += [(2**16, 1e-7, True, 2**16), (2**18 + 1, 2e-6, True, 2**17), (3001, 1e-5, False, 1000),
          (6000, 0.999, True, 7), (6000, 0.99, False, 1), (9000, 0.9999, False, 50), (700, 1.0, True, 700),
          (5000, 0.0, False, 9), (1, 0.3, True, 1)]


@pytest.mark.parametrize("n,p,directed,chunks", CASES)
def test_sparse_tiles_equal_oracle(kgref, n, p, directed, chunks):
    import torch
    kg = require_gpu()
    want = kgref.skip_generate(kgref.inst(n, p=p, directed=directed, seed=17, chunks=chunks, model=kgref.GNP))
    inst = kg.Instance(n, kg.GNP, directed, 0, p, 17, chunks)
    plain = torch.empty(kg.workspace_bytes([inst]), dtype=torch.uint8, device="cuda")
    for ws in (None, plain):
        got = kg.gnp_skip(n, p, directed, 17, chunks, workspace=ws)      # counted, then written
        torch.cuda.synchronize()
        assert got.shape[0] == len(want)
        assert np.array_equal(to_np_u32(got), want)
    out = torch.full((max(len(want) - 1, 0), 2), 7, dtype=torch.int32, device="cuda").view(torch.uint32)
    _, total = kg.gnp_skip(n, p, directed, 17, chunks, out=out, workspace=plain)
    torch.cuda.synchronize()
    assert int(to_np_u64(total)[0]) == len(want)
    assert np.all(to_np_u32(out) == 7)
