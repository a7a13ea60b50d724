"""Keyframe gradients reach the keys that they belong to and no other: one that
is not finite the two keys of its reader's frame in each clip, also where
another key shares a workgroup with them; and in libraries of more keys than a
launch has workgroups."""
import numpy as np
import pytest
import torch

from oracle.sample_backward import pose_sample_backward
from paper_2505_06703_amd import hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clips", [3, 300])  # one key a workgroup; two
@pytest.mark.parametrize("keys", [4, 5])
@pytest.mark.parametrize("workspace", [False, True])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_only_the_keys_that_it_reads(clips, keys, workspace, value):
    rng = np.random.default_rng(clips + keys)
    chars, joints = 4 * clips * keys, 5
    off = np.arange(chars + 1, dtype=np.int64) * joints
    par = np.tile(np.arange(-1, joints - 1, dtype=np.int32), chars)
    kq = rng.standard_normal((clips, keys, joints, 4)).astype(np.float32)
    kq /= np.linalg.norm(kq, axis=-1, keepdims=True)
    kt = rng.standard_normal((clips, keys, joints, 3)).astype(np.float32)
    ca, cb = np.arange(chars) % clips, (np.arange(chars) + 1) % clips
    k0 = np.arange(chars) // (4 * clips)
    fps = 32.0
    time = ((k0 + 0.375) / fps).astype(np.float32)
    gq, gt = (rng.standard_normal((chars * joints, n)).astype(np.float32) for n in (4, 3))
    hit = np.zeros((clips, keys), bool)
    bad = rng.choice(chars, 3, replace=False)
    for c in bad:
        gq[c * joints:(c + 1) * joints] = gt[c * joints:(c + 1) * joints] = value
        for clip in (ca[c], cb[c]):
            hit[clip, [k0[c], (k0[c] + 1) % keys]] = True
    plan = hs.Plan(off, par)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in
           (kq, kt, ca.astype(np.int32), cb.astype(np.int32), time, np.full(chars, 0.25, np.float32), gq, gt)]
    lib = hs.ClipLibrary(dev[0], dev[1], fps)
    ws = hs.sample_backward_workspace(plan, "cuda:0") if workspace else None
    got = hs.hs_pose_sample_backward(plan, lib, *dev[2:], workspace=ws)
    for name, g in zip(("key_quat", "key_trans"), got):
        finite = np.isfinite(g.cpu().numpy()).all(axis=(2, 3))
        np.testing.assert_array_equal(finite, ~hit, err_msg=name)


@pytest.mark.parametrize("keys", [1, 3])
@pytest.mark.parametrize("workspace", [False, True])
def test_more_keys_than_workgroups(keys, workspace):
    """Workgroups that take more than one group of keys (a launch has 2^20),
    most of them without a reader.

    Tolerance: |g_gpu - g_fp64| <= 1e-4 * max(1, max |g_fp64|), as in
    test_gpu_key_pairs.py."""
    clips, chars, joints, fps = 1200000 // ((keys + 1) // 2), 400, 2, 30.0
    rng = np.random.default_rng(keys)
    off = np.arange(chars + 1, dtype=np.int64) * joints
    used = np.unique(np.concatenate([[0, clips - 1], rng.integers(0, clips, 50)]))
    kq = rng.standard_normal((used.size, keys, joints, 4)).astype(np.float32)
    kq /= np.linalg.norm(kq, axis=-1, keepdims=True)
    kt = rng.standard_normal((used.size, keys, joints, 3)).astype(np.float32)
    ca, cb = rng.integers(0, used.size, (2, chars)).astype(np.int32)
    time = rng.uniform(-1.0, 2.0, chars).astype(np.float32)
    weight = rng.uniform(0.2, 0.8, chars).astype(np.float32)
    gq, gt = (rng.standard_normal((chars * joints, n)).astype(np.float32) for n in (4, 3))
    ref = pose_sample_backward(off, kq, kt, ca, cb, time, weight, gq, gt, fps)

    plan = hs.Plan(off, np.tile(np.array([-1, 0], np.int32), chars))
    rows = torch.from_numpy(used).cuda()
    big = [torch.ones((clips, keys, joints, n), device="cuda") for n in (4, 3)]
    for b, a in zip(big, (kq, kt)):
        b[rows] = torch.from_numpy(a).cuda()
    dev = [torch.from_numpy(a).cuda() for a in
           (used[ca].astype(np.int32), used[cb].astype(np.int32), time, weight, gq, gt)]
    ws = hs.sample_backward_workspace(plan, "cuda:0") if workspace else None
    got = hs.hs_pose_sample_backward(plan, hs.ClipLibrary(*big, fps), *dev, workspace=ws)
    for name, g, r in zip(("key_quat", "key_trans"), got, ref):
        err = np.abs(g[rows].cpu().numpy().astype(np.float64).reshape(r.shape) - r).max()
        assert err <= 1e-4 * max(1.0, np.abs(r).max()), f"{name}: {err:.3e}"
        g[rows] = 0.0
        assert not g.any(), name
