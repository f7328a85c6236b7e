"""The skip sampler on tiles of 2^32 slots with 60 to 559 expected events: one
round of 128 waiting times spans 2^30 to past 2^32 slots, so the advance to the
next round has its bit 31 set or needs a 33rd.  With stored rows, regenerated,
and the count alone, byte for byte against the oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("chunks", [1, 37])
@pytest.mark.parametrize("events", [60, 100, 128, 160, 200, 256, 300, 420, 559])
def test_wide_sums_equal_oracle(kgref, events, chunks, directed):
    import torch
    kg = require_gpu()
    n, p = 2**19 + 11, events / 2.0**32
    I = kgref.inst(n, p=p, directed=directed, seed=13, chunks=chunks, model=kgref.GNP)
    assert kgref.tile_exponent(I) == 32
    want = kgref.skip_generate(I)
    inst = kg.Instance(n, kg.GNP, directed, 0, p, 13, chunks)
    for size in (kg.gnp_skip_workspace_bytes(n, p, directed, chunks), kg.workspace_bytes([inst])):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out = torch.full((len(want), 2), 7, dtype=torch.int32, device="cuda").view(torch.uint32)
        none = torch.empty((0, 2), dtype=torch.uint32, device="cuda")
        _, total = kg.gnp_skip(n, p, directed, 13, chunks, out=none, workspace=ws)
        torch.cuda.synchronize()
        assert int(to_np_u64(total)[0]) == len(want), size
        _, total = kg.gnp_skip(n, p, directed, 13, chunks, out=out, workspace=ws)
        torch.cuda.synchronize()
        assert int(to_np_u64(total)[0]) == len(want), size
        assert np.array_equal(to_np_u32(out), want), size
