"""One step a launch with four voxels a lane against the one-thread-per-voxel
reference, bit for bit, on both forms of its damage update: planes of a
multiple of 2^14 voxels (with and without whole tiles) and others, cached and
streaming stores, with sums and a latched, damaged core."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("shape, store", [((9, 64, 256), 1), ((9, 64, 256), 3), ((5, 32, 512), 2),
                                          ((9, 20, 260), 1), ((6, 63, 256), 3), ((7, 21, 512), 2),
                                          ((5, 128, 128), 1)])
@pytest.mark.parametrize("tile_y", [4, 8])
def test_bitwise_equals_reference(shape, store, tile_y, field):
    case = W.random_tissue_case(73, shape=shape, n_classes=5, n_tines=2, n_steps=40)
    grids = []
    for kw in (dict(kernel=1), dict(kernel=2, depth=1, z_vec=4, tile_y=tile_y,
                                    store_policy=store)):
        g = rfa.Grid(case.shape, case.spacing, t_death=case.t_death, A=6.0e8, Ea=5.0e4, **kw)
        g.load_case(case)
        if field:
            g.set_perfusion(np.random.default_rng(71).uniform(0.5, 2.0, case.shape)
                            .astype(np.float32))
        # hot enough in places to be damaged and to cross the threshold on the way
        g.set_temperature(np.random.default_rng(74).uniform(37.0, 75.0, case.shape))
        grids.append(g)
    g1, g2 = grids
    plan = g2.plan()
    assert (plan["depth"], plan["z_vec"], plan["tile_y"]) == (1, 4, tile_y)
    dt = 0.9 * min(case.dt, g1.dt_max())
    for n in (1, 7, 20):
        d1, d2 = g1.step(n, dt, diag=True), g2.step(n, dt, diag=True)
        for a, b in zip(g1.raw_state(), g2.raw_state()):
            assert np.array_equal(a, b), n
        (m1, o1, _), (m2, o2, _) = g1.damage(), g2.damage()
        assert np.array_equal(m1, m2) and np.array_equal(o1, o2), n
        assert d1["mono_violations"] == d2["mono_violations"]
        assert d1["energy_J"] == d2["energy_J"]
    assert m1.any()
    for g in grids:
        g.close()
