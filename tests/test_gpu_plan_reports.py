"""What grids and batches report of their launches is what they take."""
from __future__ import annotations

import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, kw, pair", [
    ((32, 32, 32), {}, "4x1"),
    ((9, 40, 60), dict(depth=2, tile_y=8, tile_x=1), "8x"),
    ((13, 21, 255), {}, "16x2"),
    ((24, 70, 256), {}, "16x2"),
    ((9, 20, 257), dict(depth=2), None),     # rows only the 2.5-D kernel takes
    ((9, 20, 257), {}, None),
    ((32, 32, 32), dict(depth=1), None),
    ((32, 32, 32), dict(tile_x=8), None),    # a one-step shape asked for
])
def test_grid(shape, kw, pair):
    g = rfa.Grid(shape, (1e-3,) * 3, **kw)
    plan = g.plan()
    if pair is None:
        assert plan["pair"] is None
        assert plan["depth"] == kw.get("depth", 1)
    else:
        assert plan["pair"].startswith(pair) and plan["depth"] == 2
        waves, lane_voxels = map(int, plan["pair"].split("x"))
        assert (plan["tile_y"], plan["z_vec"]) == (waves, lane_voxels)
    g.close()


def test_batch():
    case = W.case_straight(n=40, n_steps=0, seed=2031)
    grids = []
    for _ in range(2):
        g = rfa.Grid(case.shape, case.spacing)
        g.load_case(case)
        grids.append(g)
    dt = 0.9 * min(case.dt, grids[0].dt_max())
    b = rfa.Batch(grids, [dt] * 2)
    plan = b.plan()
    assert plan["depth"] == 2 and plan["pair"] and plan["pair_items"] >= 2
    grids[0].set_perfusion_decay(True)  # coupled grids take one step a launch
    b.step(2)
    assert {k: b.plan()[k] for k in ("depth", "pair", "pair_items")} == dict(
        depth=1, pair=None, pair_items=0)
    grids[0].set_perfusion_decay(False)
    b.step(2)
    assert b.plan() == plan
    assert b.set_plan(tile_x=4)["depth"] == 1
    b.close()
    for g in grids:
        g.close()
