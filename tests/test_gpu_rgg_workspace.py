"""Three-dimensional graphs in workspaces that hold only what the
lane-per-vertex passes take: the same output as with the reported size, KG_ENOSPC
below it, and a call without a workspace where torch has no room for one."""
import ctypes
import math

import numpy as np
import pytest

from gpu_util import require_gpu, to_np_u32, to_np_u64


def lane_bytes(n, L):
    """The lane-per-vertex layout: first vertices and split buffers of the cells,
    24 bytes per vertex, counts and offsets per 64 vertices, scan sums, status."""
    depth, launches = 3 * L, max(1, (3 * L + 11) // 12)
    p = 0
    for i in range(launches - 1):
        p += (depth - p) // (launches - i)
    words = (1 << p) + 32 if launches > 1 else 0
    waves = (n + 63) // 64
    parts = [16 * words, 8 * (8**L + 1), 4 * n, 4 * n, 16 * n, 8 * (waves + 1), 8 * (waves + 1),
             8 * ((waves + 4095) // 4096 + 1), 32]
    return sum((b + 255) & ~255 for b in parts)


@pytest.mark.gpu
@pytest.mark.parametrize("L,a", [(3, 1.0), (3, 4.0), (4, 6.0), (4, 12.0), (0, 20.0)])
def test_smaller_workspace_same_bytes(kgref, L, a):
    import torch
    kg = require_gpu()
    n, r, seed = int(a * 8**L), 0.9 * 2.0**-L, 5
    least = lane_bytes(n, L)
    assert least < kg.rgg3d_workspace_bytes(n, r)
    want_points, want_edges = kgref.rgg3d(n, r, seed)
    for size in (least, kg.rgg3d_workspace_bytes(n, r) - 1):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out = torch.empty((len(want_edges), 2), dtype=torch.uint32, device="cuda")
        points, edges, total = kg.rgg3d(n, r, seed, out=out, workspace=ws)
        torch.cuda.synchronize()
        assert int(to_np_u64(total)[0]) == len(want_edges)
        assert np.array_equal(to_np_u32(edges), want_edges)
        assert np.array_equal(points.cpu().numpy().view(np.uint64), want_points.view(np.uint64))
    with pytest.raises(kg.KgError):
        kg.rgg3d(n, r, seed, out=out, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.gpu
@pytest.mark.parametrize("d", [2, 3])
def test_no_room_for_a_workspace(kgref, monkeypatch, d):
    import torch
    kg = require_gpu()
    name = "rgg%dd" % d
    monkeypatch.setattr(kg, name + "_workspace_bytes", lambda n, r: 1 << 50)
    points, edges = getattr(kg, name)(5000, 0.06, seed=3)
    torch.cuda.synchronize()
    assert np.array_equal(to_np_u32(edges), getattr(kgref, name)(5000, 0.06, 3)[1])


def test_reported_size_fits_the_card():
    """Points, mean edges and the reported workspace together stay below the
    card's memory where the lane-per-vertex passes' do (r = 0.55 (ln n / n)^(1/3))."""
    from paper_1710_07565_amd import _lib
    b = ctypes.c_uint64(0)
    for n in (2**26, 2**28, 2**30, 3 * 2**29, 2**31, 5 * 2**29, 2**32 - 1):
        r = 0.55 * (math.log(n) / n) ** (1.0 / 3.0)
        assert _lib.lib().kg_rgg3d_workspace_bytes(n, r, ctypes.byref(b)) == _lib.KG_OK
        rest = 24 * n + 8 * (0.5 * n * n * 4.1888 * r**3)
        L = int(math.log2(1.0 / r))
        L = min(L, 10)
        assert lane_bytes(n, L) <= b.value
        assert b.value + rest <= 288 * 2**30 or b.value == lane_bytes(n, L)
