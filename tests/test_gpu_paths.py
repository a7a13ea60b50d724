"""GPU parity of the path adjoint (the adjoint that HS_ADJ_AUTO takes for
characters of up to 1024 joints) against the FP64 oracle, at the sizes where
its pieces, waves and workgroups end: pieces of eight joints, 64 pieces a
wave, one to eight waves a workgroup.

Tolerance as for every adjoint: per character, max |grad_gpu - grad_fp64| <=
1e-4 * max(1, max |grad_fp64|) for each gradient array.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_06703_amd import hs
from paper_2505_06703_amd import workloads as wl
from parity import check_global, reference
from test_gpu_backward import check_grads, dev, oracle_grads, run

pytestmark = pytest.mark.gpu


def chain(n):
    return np.arange(-1, n - 1)


def comb(teeth, length):
    """A spine with a chain of `length` joints below each of its joints."""
    par = []
    for _ in range(teeth):
        prev = len(par) - 1 - length if par else -1
        par.append(prev)
        for _ in range(length):
            par.append(len(par) - 1)
    return np.array(par)


def fan(n, arms):
    """`arms` chains below the root."""
    par = [-1]
    for a in range(arms):
        k = (n - 1) // arms
        par += [0] + list(range(len(par), len(par) + k - 1))
    return np.array(par)


def random_tree(n, p, seed):
    rng = np.random.default_rng(seed)
    j = np.arange(n)
    par = np.where(rng.random(n) < p, j - 1, np.floor(rng.random(n) * j).astype(np.int64))
    par[0] = -1
    return par


def forest(n, roots):
    par = chain(n)
    par[:: max(1, n // roots)] = -1
    return par


TREES = {
    "one joint": [chain(1)],
    "chains at piece ends": [chain(n) for n in (2, 7, 8, 9, 15, 16, 17)],
    "one full wave": [chain(512)],
    "a wave and a joint": [chain(513)],
    "largest chain": [chain(1024)],
    "combs": [comb(30, 7), comb(30, 8), comb(31, 16), comb(100, 9)],
    "fans": [fan(513, 64), fan(129, 64), fan(1024, 33)],
    "trees of every workgroup size": [random_tree(n, p, 3) for n, p in ((60, 0.5), (300, 0.7), (700, 0.8), (1024, 0.6))],
    "forests, empty characters": [forest(200, 5), np.zeros(0, int), forest(1000, 90), np.zeros(0, int)],
    "beside larger characters": [random_tree(900, 0.8, 5), random_tree(1500, 0.8, 6), chain(40), chain(4000), chain(40)],
}


def batch(trees, seed=0, scale=True):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum([t.size for t in trees])]).astype(np.int64)
    par = np.concatenate(trees).astype(np.int32)
    q, t, s = wl.random_pose(rng, par.size)
    if scale:
        s = rng.uniform(0.95, 1.05, s.shape).astype(np.float32)
    return wl.Batch("paths", off, par, q, t, s, q, t, s)


@pytest.mark.parametrize("name", TREES)
def test_dense_seed(name):
    b = batch(TREES[name])
    W = np.random.default_rng(1).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    check_grads(b.offsets, run(b, W), oracle_grads(b, W), name)


@pytest.mark.parametrize("copies", [1, 40, 3000])
def test_small_characters_share_workgroups(copies):
    b = batch([t for _ in range(copies) for t in (chain(11), random_tree(30, 0.6, 2), chain(1))])
    W = np.random.default_rng(2).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    check_grads(b.offsets, run(b, W), oracle_grads(b, W), f"{copies} copies")


@pytest.mark.parametrize("name", [k for k in TREES if k != "beside larger characters"])
@pytest.mark.parametrize("scale", [True, False])
def test_effector_step_and_backward(name, scale):
    """Sparse seeds: every third joint (the first and last ones too), from a
    given forward output and from the kernel's own scan."""
    b = batch(TREES[name], scale=scale)
    plan = hs.Plan(b.offsets, b.parents)
    eff = np.unique(np.concatenate([np.arange(0, b.num_joints, 3), [b.num_joints - 1]]))
    y = np.random.default_rng(3).standard_normal((eff.size, 3)).astype(np.float32)
    E = hs.Effectors(plan, eff)
    assert E.sparse
    q, t, s = dev(b.quat), dev(b.trans), dev(b.scale) if scale else None
    Gr, lam, _ = reference(b)
    seed = np.zeros((b.num_joints, 4, 4))
    seed[eff, :3, 3] = 2.0 * (Gr[eff, :3, 3] - y)
    ref = oracle.backward(b.offsets, b.parents, b.quat, b.trans, b.scale, seed)
    G = torch.empty((b.num_joints, 4, 4), device="cuda:0")
    got = hs.hs_effector_step(plan, E, q, t, s, dev(y), global_out=G)
    check_global(G.cpu().numpy(), Gr, lam, name)
    check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, f"{name}, step")
    got = hs.hs_effector_step(plan, E, q, t, s, dev(y))
    check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, f"{name}, step without G")
    got = hs.hs_effector_backward(plan, E, q, t, s, G, dev(y))
    check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, f"{name}, backward")
    E.close()


def test_no_seed_below_a_joint_that_is_not_finite():
    """A pose that is not finite spoils only the gradients that its
    transform enters: effectors of another character keep theirs."""
    b = batch([chain(300), chain(300)])
    plan = hs.Plan(b.offsets, b.parents)
    eff = np.array([299, 599])
    y = np.zeros((2, 3), np.float32)
    E = hs.Effectors(plan, eff)
    q = b.quat.copy()
    q[450] = np.nan
    ref = hs.hs_effector_step(plan, E, dev(b.quat), dev(b.trans), dev(b.scale), dev(y))
    got = hs.hs_effector_step(plan, E, dev(q), dev(b.trans), dev(b.scale), dev(y))
    assert torch.equal(got[0][:300], ref[0][:300])
    assert torch.isnan(got[0][599]).all()
    E.close()
