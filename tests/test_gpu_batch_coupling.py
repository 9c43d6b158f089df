"""Damage-coupled perfusion switched on and off in a live batch, with calls on
the grid itself in between that renew its tables: every launch form of the
batch (two steps, one step) equals grids stepped alone by the reference
kernel, bit for bit."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


def _grids(cases, **kw):
    out = []
    for k, c in enumerate(cases):
        g = rfa.Grid(c.shape, c.spacing, A=6.0e8, Ea=5.0e4, **kw)
        g.load_case(c)
        # a field of its own, so that switching the coupling allocates nothing
        g.set_perfusion(np.random.default_rng(90 + k).uniform(0.5, 2.0, c.shape)
                        .astype(np.float32))
        out.append(g)
    return out


def _same(alone, batched, what):
    for i, (g1, g2) in enumerate(zip(alone, batched)):
        for a1, a2 in zip(g1.raw_state(), g2.raw_state()):
            assert np.array_equal(a1, a2), (what, i)
        assert np.array_equal(g1.omega(), g2.omega()), (what, i)


@pytest.mark.parametrize("between", [0, 4])
@pytest.mark.parametrize("first", [False, True])
def test_coupling_switched_in_a_live_batch(between, first):
    cases = [dataclasses.replace(W.random_tissue_case(30 + i, shape=s, n_classes=4, n_tines=2),
                                 perfusion_decay=False)
             for i, s in enumerate([(26, 33, 40), (20, 24, 31)])]
    alone, batched = _grids(cases, kernel=1), _grids(cases)
    dts = [0.9 * min(c.dt, g.dt_max()) for c, g in zip(cases, alone)]
    for g in (alone[0], batched[0]):
        g.set_perfusion_decay(first)
    b = rfa.Batch(batched, dts)
    on = first
    for n in (6, 9, 6, 9):
        b.step(n)
        for g, dt in zip(alone, dts):
            g.step(n, dt, diag=False)
        _same(alone, batched, (on, n))
        on = not on
        for g in (alone[0], batched[0]):
            g.set_perfusion_decay(on)
            g.step(between, dts[0], diag=False)
    # the coupling acted: the same steps without it end elsewhere
    never = _grids(cases[:1], kernel=1)
    never[0].step(alone[0].step_count(), dts[0], diag=False)
    assert not np.array_equal(never[0].temperature(), alone[0].temperature())
    b.close()
    for g in alone + batched + never:
        g.close()


@pytest.mark.parametrize("shape", [(26, 33, 40), (9, 20, 260)])
def test_tuning_a_coupled_grid_in_a_live_batch(shape):
    """Tuning times the coupled launches on scratch images of their own and
    leaves state and batch as they were."""
    case = dataclasses.replace(W.random_tissue_case(33, shape=shape, n_classes=4, n_tines=2),
                               perfusion_decay=False)
    (alone,), (grid,) = _grids([case], kernel=1), _grids([case])
    dt = 0.9 * min(case.dt, alone.dt_max())
    b = rfa.Batch([grid], [dt])
    for g in (alone, grid):
        g.set_perfusion_decay(True)
    grid.tune(dt, reps=2)
    for n in (7, 6):
        alone.step(n, dt, diag=False)
        b.step(n)
        _same([alone], [grid], n)
        alone.step(n, dt, diag=False)
        grid.step(n, dt, diag=False)
        _same([alone], [grid], n)
        grid.tune(dt, reps=2)
    b.close()
    for g in (alone, grid):
        g.close()
