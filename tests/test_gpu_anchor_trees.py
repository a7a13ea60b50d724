"""GPU parity of the multipass path for branched characters, whose anchors
are taken level by level (at most 64 levels, 3072 anchors a character) or in
rounds of pointer jumping beyond: forward and adjoint against the FP64 oracle
on both sides of those lines.

Tolerances as for every forward and adjoint (parity.py, test_gpu_backward.py).
"""
import numpy as np
import pytest

from paper_2505_06703_amd import hs
from paper_2505_06703_amd import workloads as wl
from parity import check_global, reference
from test_gpu_backward import check_grads, dev, oracle_grads, run

pytestmark = pytest.mark.gpu


def tree(n, p, seed):
    rng = np.random.default_rng(seed)
    j = np.arange(n)
    par = np.where(rng.random(n) < p, j - 1, np.floor(rng.random(n) * j).astype(np.int64))
    par[0] = -1
    return par


def star(n):
    par = np.zeros(n, np.int64)
    par[0] = -1
    return par


def run_of_blocks(levels, extra=0):
    """A chain through `levels` + 1 blocks of 64 joints (an anchor at the end
    of each but the last), two more joints below the first joint making it
    branched, `extra` joints below the last one."""
    n = 64 * (levels + 1)
    par = np.arange(-1, n - 1)
    return np.concatenate([par, [0, 0], np.full(extra, n - 1)])


def every_block_its_own(blocks):
    """Blocks of 64 joints, each a chain below joint 64 b + 5 of an earlier block."""
    par = []
    for b in range(blocks):
        par += [-1 if b == 0 else 64 * (b // 2) + 5] + list(range(64 * b, 64 * b + 63))
    return np.array(par)


CASES = {
    "a star: one anchor": [star(4000)],
    "forest of big trees": [np.concatenate([tree(2500, 0.9, 1), np.where(tree(700, 0.8, 2) < 0, -1, tree(700, 0.8, 2) + 2500)])],
    "binary tree of blocks": [every_block_its_own(63)],
    "64 levels": [run_of_blocks(64)],
    "65 levels": [run_of_blocks(65)],
    "beside small ones and chains": [tree(3000, 0.95, 3), tree(50, 0.7, 4), np.arange(-1, 4999), tree(9000, 0.97, 5)],
    "anchors at the limit": [tree(8000, 0.45, 6), tree(7000, 0.45, 7)],
    "anchors beyond it": [tree(30000, 0.3, 8)],
}


def batch(trees, seed=0):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum([t.size for t in trees])]).astype(np.int64)
    par = np.concatenate(trees).astype(np.int32)
    q, t, s = wl.random_pose(rng, par.size, max_angle=0.05)
    s = rng.uniform(0.99, 1.01, s.shape).astype(np.float32)
    return wl.Batch("big", off, par, q, t, s, q, t, s)


@pytest.mark.parametrize("name", CASES)
def test_forward_and_adjoint(name):
    b = batch(CASES[name])
    plan = hs.Plan(b.offsets, b.parents)
    assert plan.info["multipass_joints"] > 0
    Gr, lam, _ = reference(b)
    q, t, s = dev(b.quat), dev(b.trans), dev(b.scale)
    for _ in range(2):
        G, _ = hs.hs_scan_forward(plan, q, t, s)
        check_global(G.cpu().numpy(), Gr, lam, name)
    W = np.random.default_rng(1).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    ref = oracle_grads(b, W)
    for _ in range(2):
        got = hs.hs_scan_backward(plan, q, t, s, dev(W))
        check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, name)


def test_small_characters_on_the_multipass_path():
    b = batch([tree(n, 0.7, n) for n in (1, 63, 64, 65, 300, 1000)])
    W = np.random.default_rng(2).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    check_grads(b.offsets, run(b, W, strategy=hs.HS_STRATEGY_MULTIPASS), oracle_grads(b, W), "multipass")
