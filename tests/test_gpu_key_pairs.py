"""Keyframe gradients at the edges of their gather: one or two keys a
workgroup (two from 256 pairs of keys on), clips of one, two and odd numbers
of keys, lists longer than one round, more characters than one segment of the
scan, more joints than a workgroup has threads, empty characters; with and
without a workspace, against the FP64 oracle.

Tolerance: |g_gpu - g_fp64| <= 1e-4 * max(1, max |g_fp64|).  A key's value is
an fp32 sum of n terms of random sign and about unit size: it grows as
sqrt(n), its rounding as sqrt(n) u times its size (u = 6e-8), which at the
n <= 30 000 here is 1e-5 of it; a term's own error is some tens of u.
"""
import numpy as np
import pytest
import torch

from oracle.sample_backward import pose_sample_backward
from paper_2505_06703_amd import hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clips, keys, chars, joints, one_clip", [
    (1, 1, 40, 5, False),
    (1, 2, 40, 300, False),
    (2, 3, 20000, 2, False),
    (255, 2, 300, 70, False),
    (256, 1, 300, 70, False),
    (256, 2, 1500, 9, True),
    (128, 3, 400, 300, False),
    (256, 2, 20000, 2, True),
])
def test_key_gradients(clips, keys, chars, joints, one_clip):
    rng = np.random.default_rng(clips * 7 + keys)
    sizes = rng.integers(0, joints + 1, chars)
    sizes[0], sizes[-1] = joints, 0
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    par = np.concatenate([np.arange(n) - 1 for n in sizes]).astype(np.int32)
    N = int(off[-1])

    def normal(*shape):
        return rng.standard_normal(shape).astype(np.float32)

    kq = normal(clips, keys, joints, 4)
    kq /= np.linalg.norm(kq, axis=-1, keepdims=True)
    kt = normal(clips, keys, joints, 3)
    ca = np.full(chars, clips // 2, np.int32) if one_clip else rng.integers(0, clips, chars).astype(np.int32)
    cb = rng.integers(0, clips, chars).astype(np.int32)
    time = rng.uniform(-1.0, 2.0, chars).astype(np.float32)
    weight = rng.uniform(0.2, 0.8, chars).astype(np.float32)
    gq, gt, fps = normal(N, 4), normal(N, 3), 30.0
    ref = pose_sample_backward(off, kq, kt, ca, cb, time, weight, gq, gt, fps)

    plan = hs.Plan(off, par)
    kq, kt, ca, cb, time, weight, gq, gt = (torch.from_numpy(a).cuda() for a in (kq, kt, ca, cb, time, weight, gq, gt))
    lib = hs.ClipLibrary(kq, kt, fps)
    for what, ws in (("no workspace", None), ("workspace", hs.sample_backward_workspace(plan, "cuda:0"))):
        got = hs.hs_pose_sample_backward(plan, lib, ca, cb, time, weight, gq, gt, workspace=ws)
        for name, g, r in zip(("key_quat", "key_trans"), got, ref):
            err = np.abs(g.cpu().numpy().astype(np.float64).reshape(r.shape) - r).max()
            assert err <= 1e-4 * max(1.0, np.abs(r).max()), f"{name}, {what}: {err:.3e}"
