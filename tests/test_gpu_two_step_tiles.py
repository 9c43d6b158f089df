"""The 2.5-D two-step kernel, which takes rows beyond the flat two-step
kernel's 256 voxels, against the one-thread-per-voxel reference, bit for bit:
ragged tiles, rows just over the limit and over several tiles, odd and even
step counts, chunk lengths of 2 mod 4 planes and others; and the calls that
fall back to one step a launch there."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pair_of_grids(case, ty, xc, field=False, coupled=False):
    grids = []
    for kw in (dict(kernel=1), dict(kernel=2, depth=2, tile_y=ty, tile_x=xc)):
        g = rfa.Grid(case.shape, case.spacing, t_death=case.t_death, A=6.0e8, Ea=5.0e4, **kw)
        g.load_case(case)
        if field:
            g.set_perfusion(np.random.default_rng(71).uniform(0.5, 2.0, case.shape)
                            .astype(np.float32))
        g.set_perfusion_decay(coupled)
        grids.append(g)
    plan = grids[1].plan()
    assert (plan["depth"], plan["pair"]) == (2, None)  # this kernel, not the flat one
    assert (plan["tile_y"], plan["tile_x"]) == (ty, min(xc, case.shape[0]))
    return grids


def _same(g1, g2, what):
    for a, b in zip(g1.raw_state(), g2.raw_state()):
        assert np.array_equal(a, b), what
    (m1, o1, _), (m2, o2, _) = g1.damage(), g2.damage()
    assert np.array_equal(m1, m2) and np.array_equal(o1, o2), what


def _case(shape, seed=72):
    return W.random_tissue_case(seed, shape=shape, n_classes=5, n_tines=2, n_steps=40)


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("shape, ty, xc", [((9, 20, 258), 8, 4), ((9, 20, 258), 16, 6),
                                           ((14, 21, 300), 8, 14), ((14, 21, 300), 16, 5),
                                           ((5, 33, 373), 16, 2), ((7, 5, 257), 8, 7)])
def test_bitwise_equals_reference(shape, ty, xc, field):
    case = _case(shape)
    g1, g2 = _pair_of_grids(case, ty, xc, field)
    dt = 0.9 * min(case.dt, g1.dt_max())
    for n in (1, 2, 6, 33):
        d1, d2 = g1.step(n, dt, diag=True), g2.step(n, dt, diag=True)
        _same(g1, g2, n)
        assert d1["mono_violations"] == d2["mono_violations"]
        assert d1["energy_J"] == d2["energy_J"]
        scale = abs(d1["injected_J"]) + abs(d1["perfusion_J"]) + abs(d1["boundary_J"])
        for k in ("perfusion_J", "boundary_J"):
            # FP32 sums of up to 2^20 terms in another order
            assert abs(d1[k] - d2[k]) <= 1e-6 * scale, k
    for g in (g1, g2):
        g.close()


def test_coupled_steps_take_one_step_a_launch():
    case = _case((9, 20, 258))
    g1, g2 = _pair_of_grids(case, 8, 6, field=True, coupled=True)
    dt = 0.9 * min(case.dt, g1.dt_max())
    for n in (1, 6, 33):
        for g in (g1, g2):
            g.step(n, dt, diag=False)
        _same(g1, g2, n)
    for g in (g1, g2):  # and two again once the coupling is off
        g.set_perfusion_decay(False)
        g.step(8, dt, diag=False)
    _same(g1, g2, "off")
    for g in (g1, g2):
        g.close()


@pytest.mark.parametrize("every", [0, 4])
def test_kept_and_recomputed_trajectories(every):
    """Kept images (one step a launch) and, with checkpoints, segments of two
    steps a launch that the adjoint recomputes in single ones."""
    case = _case((9, 20, 258))
    out = []
    for g in _pair_of_grids(case, 8, 6):
        dt = 0.9 * min(case.dt, g.dt_max())
        g.forward_checkpointed(11, dt, every)
        w = np.random.default_rng(4).uniform(0.5, 1.0, case.shape).astype(np.float32)
        dP, _, dperf = g.adjoint(w, len(case.needle.power), 0, want_dperf=True)
        out.append((*g.raw_state(), g.omega(), dP, dperf))
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert np.abs(out[0][3]).max() > 0
