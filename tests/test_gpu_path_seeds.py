"""The path adjoint with end-effector seeds.  HS_ADJ_AUTO takes it once the
tiles of the two-level adjoint are too many to be resident at once, so every
batch here has more of them.
"""
import numpy as np
import pytest
import torch

from paper_2505_06703_amd import hs
from paper_2505_06703_amd import workloads as wl
from test_gpu_backward import dev
from test_gpu_paths import chain

pytestmark = pytest.mark.gpu


def copies(trees, n, seed=0):
    """n characters cycling over the trees, each with a pose of its own."""
    trees = [trees[i % len(trees)] for i in range(n)]
    off = np.concatenate([[0], np.cumsum([t.size for t in trees])]).astype(np.int64)
    par = np.concatenate(trees).astype(np.int32)
    rng = np.random.default_rng(seed)
    q, t, s = wl.random_pose(rng, par.size)
    s = rng.uniform(0.95, 1.05, s.shape).astype(np.float32)
    return wl.Batch("seeds", off, par, q, t, s, q, t, s)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("where", ["quat", "trans", "scale"])
def test_a_pose_that_is_not_finite_below_every_seed(value, where):
    """Joints above it have a gradient of their own seeds alone: bitwise what
    it is with a finite pose there, at every place of the joint in its piece.
    (The transforms of what hangs below are not finite, and so neither are
    their gradients.)"""
    C, n, seeded = 800, 512, 20
    b = copies([chain(n)], C)
    bad = n * np.arange(C) + 440 + np.arange(C) % 8
    eff = b.offsets[:-1] + seeded
    y = np.random.default_rng(1).standard_normal((C, 3)).astype(np.float32)
    plan = hs.Plan(b.offsets, b.parents)
    E = hs.Effectors(plan, eff)
    assert E.sparse
    pose = {"quat": b.quat, "trans": b.trans, "scale": b.scale}
    spoilt = dict(pose, **{where: pose[where].copy()})
    spoilt[where][bad] = value
    above = np.zeros(C * n, bool)
    for o, e in zip(b.offsets[:-1], bad):
        above[o:e] = True
    above = dev(above)
    grads = []
    for p in (pose, spoilt):
        p = [dev(p[k]) for k in ("quat", "trans", "scale")]
        G, _ = hs.hs_scan_forward(plan, *p)
        grads.append((hs.hs_effector_step(plan, E, *p, dev(y)), hs.hs_effector_backward(plan, E, *p, G, dev(y))))
    for call, want, got in zip(("step", "backward"), *grads):
        for name, w, g in zip(("quat", "trans", "scale"), want, got):
            assert torch.isfinite(w).all()
            assert torch.equal(g[above], w[above]), f"{call}: gradient of {name}"
    E.close()
