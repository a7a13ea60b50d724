"""GPU parity of the multipass path on both sides of the lines between its ways
over the anchors: level by level, in segments (rounds in LDS), in rounds over
all; the adjoint changes from levels to segments beyond 48 levels where hardly
two anchors send to the same one, the forward takes segments where there are
any.

Tolerances as for every forward and adjoint (parity.py, test_gpu_backward.py).
"""
import numpy as np
import pytest

from paper_2505_06703_amd import hs
from parity import check_global, reference
from test_gpu_anchor_trees import batch, run_of_blocks, tree
from test_gpu_backward import check_grads, dev, oracle_grads

pytestmark = pytest.mark.gpu


def spine(blocks, sides):
    """A chain through `blocks` blocks of 64 joints, and `sides` more chains of
    two blocks below the end of each."""
    par = list(range(-1, 64 * blocks - 1))
    for end in range(63, 64 * blocks, 64):
        for _ in range(sides):
            par += [end] + list(range(len(par), len(par) + 127))
    return np.array(par)


CASES = {
    "48 levels, unbranched": [run_of_blocks(48)],
    "49 levels, unbranched": [run_of_blocks(49)],
    "49 levels, branched": [spine(49, 1)],
    "64 levels, branched": [spine(63, 1)],
    "64 levels, no segment": [spine(63, 18)],
    "unbranched beside branched": [run_of_blocks(60)] + [tree(3500, 0.95, k) for k in range(6)],
    "one character deeper than 64": [run_of_blocks(80)] + [tree(3500, 0.95, k) for k in range(6)],
    "adjoint alone": [tree(1800, 0.9, 1), tree(1900, 0.95, 2)],
}


@pytest.mark.parametrize("name", CASES)
def test_forward_and_adjoint(name):
    b = batch(CASES[name])
    plan = hs.Plan(b.offsets, b.parents)
    assert (plan.info["multipass_joints"] > 0) == (name != "adjoint alone")
    Gr, lam, _ = reference(b)
    q, t, s = dev(b.quat), dev(b.trans), dev(b.scale)
    W = np.random.default_rng(1).standard_normal((b.num_joints, 4, 4)).astype(np.float32)
    ref = oracle_grads(b, W)
    for _ in range(2):
        G, _ = hs.hs_scan_forward(plan, q, t, s)
        check_global(G.cpu().numpy(), Gr, lam, name)
        got = hs.hs_scan_backward(plan, q, t, s, dev(W))
        check_grads(b.offsets, [g.cpu().numpy() for g in got], ref, name)
