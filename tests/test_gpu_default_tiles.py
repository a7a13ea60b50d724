"""Default tiles at the edges of their rule (a capacity of the largest
character's size, at least 256 joints): batches large enough for several
tiles per compute unit, with characters that fill a tile, miss it by one or
need one of their own, on ordinary and instanced plans."""
import numpy as np
import pytest
import torch

from paper_2505_06703_amd import hs
from paper_2505_06703_amd import workloads as wl

from parity import check_global, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1, 63, 64, 128, 255, 256, 257, 1024, 1025])
def test_default_tiles(size):
    rng = np.random.default_rng(size)
    par = np.array([-1] + [j - 1 if rng.uniform() < 0.7 else rng.integers(0, j) for j in range(1, size)], np.int32)
    C = 140000 // size + 1  # more than 512 joints for each of 256 compute units
    off = np.arange(C + 1, dtype=np.int64) * size
    allpar = np.tile(par, C)
    q, t, s = wl.random_pose(rng, C * size)
    s = rng.uniform(0.9, 1.1, s.shape).astype(np.float32)
    pose = [torch.from_numpy(a).cuda() for a in (q, t, s)]
    b = wl.Batch("copies", off, allpar, q, t, s, q, t, s)
    Gr, lam, _ = reference(b)
    G = {}
    for name, plan in (("queue", hs.Plan(off, allpar)),
                       ("classes", hs.Plan(off, allpar, schedule=hs.HS_SCHED_CLASSES)),
                       ("instanced", hs.Plan.instanced(off[:2], par, np.zeros(C, np.int32)))):
        assert plan.info["tile_joints"] == max(256, -(-size // 64) * 64)
        G[name] = hs.hs_scan_forward(plan, *pose)[0].cpu().numpy()
        check_global(G[name], Gr, lam, name)
    np.testing.assert_array_equal(G["instanced"], G["classes"])
