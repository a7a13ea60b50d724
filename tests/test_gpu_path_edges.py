"""GPU parity of the path adjoint against the FP64 oracle where its pieces (up
to four joints), waves (64 pieces), workgroups (one, two, up to four, up to
eight waves) and tables (64 pieces below a joint, 512 in a character) end, for
dense seeds and for end effectors, whose adjoint it runs from its own scan or
from a given forward.

Batches are large enough for HS_ADJ_AUTO to take it: more than four tiles of
the rounds for each compute unit, or trees whose sends contend there, and more
tiles than the two-level adjoint keeps resident at once.

Tolerances as for every forward and adjoint (parity.py, test_gpu_backward.py).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_06703_amd import hs
from parity import check_global, reference
from test_gpu_backward import check_grads, dev, oracle_grads
from test_gpu_path_seeds import copies
from test_gpu_paths import chain, comb, fan, forest, random_tree

pytestmark = pytest.mark.gpu


def comb_and_chain(teeth, length):
    """A spine with a leaf below each of its joints, and a chain at its end."""
    par = []
    for k in range(teeth):
        par += [2 * k - 2 if k else -1, 2 * k]
    return np.array(par + [2 * teeth - 2] + list(range(2 * teeth, 2 * teeth + length - 1)))


def pieces(par):
    """Pieces of at most four joints: a path goes on to the child with the most levels below it."""
    height, best, at, count = np.ones(par.size, int), np.full(par.size, -1), np.zeros(par.size, int), 0
    for j in range(par.size - 1, 0, -1):
        p = par[j]
        if p >= 0 and height[j] + 1 >= height[p]:
            height[p], best[p] = height[j] + 1, j
    for j, p in enumerate(par):
        at[j] = (at[p] + 1) % 4 if p >= 0 and best[p] == j else 0
        count += at[j] == 0
    return count


# name: trees, characters that cycle over them
BATCHES = {
    "pieces": ([chain(n) for n in (3, 4, 5, 7, 8, 9, 63, 64, 65)], 16000),
    "a wave and less": ([chain(256), chain(255), chain(130), random_tree(150, 0.9, 1), forest(140, 5)], 1320),
    "a wave and a piece": ([chain(257), chain(256), random_tree(300, 0.8, 2)], 1300),
    "up to four waves": ([chain(1024), chain(1021), random_tree(500, 0.8, 3), comb(30, 7)], 1500),
    "up to eight waves": ([random_tree(1000, 0.8, 4), random_tree(1024, 0.6, 5)], 320),
    "64 pieces below a joint": ([fan(521, 65)], 600),
    "512 pieces": ([comb_and_chain(341, 340)], 320),
    "forests, empty characters": ([forest(200, 5), np.zeros(0, int), forest(250, 25), np.zeros(0, int)], 6000),
    "ragged sizes": ([random_tree(n, 0.75, n) for n in (1, 17, 40, 41, 90, 130, 200, 310)], 6000),
    # not on the path adjoint at all
    "65 pieces below a joint": ([fan(529, 66)], 600),
    "513 pieces": ([comb_and_chain(345, 326)], 320),
}


def test_sizes():
    assert pieces(comb_and_chain(341, 340)) == 512 and pieces(comb_and_chain(345, 326)) == 513
    assert pieces(chain(256)) == 64 and pieces(chain(257)) == 65


@pytest.mark.parametrize("name", BATCHES)
def test_dense_seeds(name):
    b = copies(*BATCHES[name])
    W = np.random.default_rng(1).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    plan = hs.Plan(b.offsets, b.parents)
    got = hs.hs_scan_backward(plan, dev(b.quat), dev(b.trans), dev(b.scale), dev(W))
    check_grads(b.offsets, [g.cpu().numpy() for g in got], oracle_grads(b, W), name)


@pytest.mark.parametrize("name, scale", [(n, True) for n in BATCHES] + [("ragged sizes", False)])
def test_effectors(name, scale):
    b = copies(*BATCHES[name])
    if not scale:
        b.scale[:] = 1.0
    plan = hs.Plan(b.offsets, b.parents)
    eff = np.unique(np.concatenate([np.arange(0, b.num_joints, 3), [b.num_joints - 1]]))
    y = np.random.default_rng(3).standard_normal((eff.size, 3)).astype(np.float32)
    E = hs.Effectors(plan, eff)
    assert E.sparse
    pose = dev(b.quat), dev(b.trans), dev(b.scale) if scale else None
    Gr, lam, _ = reference(b)
    seed = np.zeros((b.num_joints, 4, 4))
    seed[eff, :3, 3] = 2.0 * (Gr[eff, :3, 3] - y)
    ref = oracle.backward(b.offsets, b.parents, b.quat, b.trans, b.scale, seed)
    G = torch.empty((b.num_joints, 4, 4), device="cuda:0")
    got = hs.hs_effector_step(plan, E, *pose, dev(y), global_out=G)
    check_global(G.cpu().numpy(), Gr, lam, name)
    check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, f"{name}, step")
    again = hs.hs_effector_step(plan, E, *pose, dev(y))
    check_grads(b.offsets, [g.cpu().numpy() for g in again], ref, f"{name}, step without G")
    got = hs.hs_effector_backward(plan, E, *pose, G, dev(y))
    check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, f"{name}, backward")
    E.close()
