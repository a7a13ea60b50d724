"""The path adjoint's seeds: which of them HS_ADJ_AUTO gives to it, and a
pose that is not finite below all end effectors.  With end-effector seeds it
runs only once the tiles of the two-level adjoint are too many to be resident
at once, so those batches have more of them.

Tolerance as for every adjoint (test_gpu_backward.py).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_06703_amd import hs
from paper_2505_06703_amd import workloads as wl
from test_gpu_backward import check_grads, dev, oracle_grads
from test_gpu_paths import chain, random_tree

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


def kary(n, arity):
    return (np.arange(n) - 1) // arity


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


# chains: no two sends of the rounds meet, so their results have the same bits every time
@pytest.mark.parametrize("joints, characters, paths", [
    (5, 3, False), (32, 300, False), (32, 20000, False), (33, 20000, True), (250, 100, False), (250, 1400, True),
    (1024, 1100, True)])
def test_dense_seeds(joints, characters, paths):
    b = copies([chain(joints)], characters)
    W = np.random.default_rng(1).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    pose = dev(b.quat), dev(b.trans), dev(b.scale)
    auto, rounds = (hs.hs_scan_backward(hs.Plan(b.offsets, b.parents, adjoint=a), *pose, dev(W))
                    for a in (hs.HS_ADJ_AUTO, hs.HS_ADJ_ROUNDS))
    assert same(auto, rounds) != paths
    check_grads(b.offsets, [g.cpu().numpy() for g in auto], oracle_grads(b, W), f"{characters} x {joints}")


# one effector a character: no two sends of the two-level kernel meet
@pytest.mark.parametrize("trees, characters, step, backward", [
    ([chain(250)], 200, False, False),
    ([chain(250)], 1400, True, True),
    ([random_tree(250, 0.8, k) for k in range(5)], 3000, True, True),
    ([kary(250, 8)], 3000, False, False),     # a thread a joint
    ([kary(300, 3)], 2000, False, True),
    ([kary(61, 60)], 9000, False, False),     # stars
])
def test_effector_seeds(trees, characters, step, backward):
    b = copies(trees, characters)
    eff = b.offsets[1:] - 1
    y = np.random.default_rng(2).standard_normal((characters, 3)).astype(np.float32)
    pose = dev(b.quat), dev(b.trans), dev(b.scale)
    got = []
    for a in (hs.HS_ADJ_AUTO, hs.HS_ADJ_ANCHORS):
        plan = hs.Plan(b.offsets, b.parents, adjoint=a)
        E = hs.Effectors(plan, eff)
        G = torch.empty((b.num_joints, 4, 4), device="cuda:0")
        got.append((hs.hs_effector_step(plan, E, *pose, dev(y), global_out=G),
                    hs.hs_effector_backward(plan, E, *pose, G, dev(y))))
        E.close()
    assert same(got[0][0], got[1][0]) != step
    assert same(got[0][1], got[1][1]) != backward
    seed = np.zeros((b.num_joints, 4, 4))
    seed[eff, :3, 3] = 2.0 * (oracle.forward(b.offsets, b.parents, b.quat, b.trans, b.scale)[eff, :3, 3] - y)
    ref = oracle.backward(b.offsets, b.parents, b.quat, b.trans, b.scale, seed)
    for call, grads in zip(("step", "backward"), got[0]):
        check_grads(b.offsets, [g.cpu().numpy() for g in grads], ref, call)


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
