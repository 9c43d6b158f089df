"""The one-step tiles with a perfusion field, in launches of many waves and of
few (two builds of the kernel), against the one-thread-per-voxel reference,
bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coupled", [False, True])
@pytest.mark.parametrize("tile_x", [1, 64])
@pytest.mark.parametrize("tile_y", [4, 8, 16])
def test_bitwise_equals_reference(tile_y, tile_x, coupled):
    case = W.random_tissue_case(75, shape=(70, 130, 67), n_classes=5, n_tines=2, n_steps=40)
    rng = np.random.default_rng(76)
    field = rng.uniform(0.5, 2.0, case.shape).astype(np.float32)
    hot = rng.uniform(37.0, 75.0, case.shape)
    grids = []
    for kw in (dict(kernel=1), dict(kernel=2, depth=1, z_vec=1, tile_y=tile_y, tile_x=tile_x)):
        g = rfa.Grid(case.shape, case.spacing, t_death=case.t_death, A=6.0e8, Ea=5.0e4, **kw)
        g.load_case(case)
        g.set_perfusion(field)
        g.set_perfusion_decay(coupled)
        g.set_temperature(hot)
        grids.append(g)
    g1, g2 = grids
    plan = g2.plan()
    assert (plan["depth"], plan["z_vec"], plan["tile_y"], plan["tile_x"]) == (1, 1, tile_y, tile_x)
    # on either side of 4096 waves
    assert (plan["workgroups"] * tile_y > 4096) == (tile_x == 1)
    dt = 0.9 * min(case.dt, g1.dt_max())
    for n in (1, 6):
        d1, d2 = g1.step(n, dt, diag=True), g2.step(n, dt, diag=True)
        for a, b in zip(g1.raw_state(), g2.raw_state()):
            assert np.array_equal(a, b), n
        (m1, o1, _), (m2, o2, _) = g1.damage(), g2.damage()
        assert np.array_equal(m1, m2) and np.array_equal(o1, o2), n
        assert d1["mono_violations"] == d2["mono_violations"]
    for g in grids:
        g.close()
