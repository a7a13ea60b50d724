"""Entries of a tuning cache are found again by batches whose default tiles
are narrower than those that the entry's key was written for: the key names a
batch by its block chains on tiles of N / (2 x compute units) joints, at most
1024, whatever the default has become.
"""
import json

import numpy as np
import pytest

from paper_2505_06703_amd import hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("joints, characters, key", [
    # five blocks in a row where a character starts inside a block (512-joint
    # tiles), four on 256-joint tiles
    (250, 1000, "gfx950|N18|maxc256|chain3|chars10|inst0|strat0|sched0"),
    # nine on 1024-joint tiles, eight on 512-joint tiles
    (510, 2000, "gfx950|N20|maxc512|chain4|chars11|inst0|strat0|sched0"),
    # tiles that were not narrowed
    (250, 20, "gfx950|N13|maxc256|chain2|chars5|inst0|strat0|sched0"),
])
def test_a_stored_shape_is_found(tmp_path, joints, characters, key):
    path = tmp_path / "tune.json"
    shape = {"tile_cap": 1024, "waves": 8, "grid_per_cu": 0, "chain_units": 0, "queue_waves": 2}
    path.write_text(json.dumps({"version": 1, "entries": {key: shape}}))
    ctx = hs.Context(0)
    ctx.load_tuning(path)
    off = np.arange(characters + 1, dtype=np.int64) * joints
    par = np.tile(np.arange(-1, joints - 1, dtype=np.int32), characters)
    plan = hs.Plan(off, par, ctx=ctx, autotune=True)
    assert (plan.info["tile_joints"], plan.info["waves_per_tile"]) == (1024, 2)
    ctx.save_tuning(path)
    assert list(json.loads(path.read_text())["entries"]) == [key]
    plan.close()
    ctx.close()
