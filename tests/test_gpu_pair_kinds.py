"""Every kind of work-group of the flat two-step kernels as the automatic
plans take it, steps and gradients, without a perfusion field (waves with
scalar coefficients) and with one: bit for bit the reference kernels'.  The
kind is asserted, so that new constants of the launch model cannot leave one
untested unnoticed."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu

KINDS = [((32, 32, 32), "4x1"), ((40, 44, 44), "8x1"), ((64, 64, 64), "8x1"),
         ((64, 61, 67), "8x1"), ((60, 51, 64), "8x2"), ((61, 64, 97), "8x2"),
         ((24, 70, 256), "16x2"), ((13, 21, 255), "16x2")]


def _grids(shape, kind, field):
    rng = np.random.default_rng(8)
    sp = (1e-3, 0.9e-3, 1.1e-3)
    labels, _ = W.tissue_labels(rng, shape, sp, (0.0, 0.0, 0.0), 4e-3, 2)
    needle = W.straight_needle([0.0, 0.0, 2e-3], [0.2, 0.1, 1.0], 4e-3, 25.0, 1e-3)
    case = W.Case("regions", shape, sp, labels, W.standard_tissue(), needle, 0.04, 0, 8)
    grids = [rfa.Grid(shape, sp, kernel=1), rfa.Grid(shape, sp)]
    for g in grids:
        g.load_case(case)
        if field:
            g.set_perfusion(np.random.default_rng(3).uniform(0.5, 2.0, shape).astype(np.float32))
    assert grids[1].plan()["pair"] == kind
    return grids, 0.9 * min(case.dt, grids[0].dt_max()), needle.n_tines


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("shape, kind", KINDS)
def test_steps(shape, kind, field):
    grids, dt, _ = _grids(shape, kind, field)
    for n, diag in ((2, False), (5, True), (24, False)):
        for g in grids:
            g.step(n, dt, diag=diag)
        for a, b in zip(grids[0].raw_state(), grids[1].raw_state()):
            assert np.array_equal(a, b), n
        assert np.array_equal(grids[0].omega(), grids[1].omega()), n
    assert grids[0].temperature().max() > 45.0
    for g in grids:
        g.close()


@pytest.mark.parametrize("every", [0, 5])
@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("shape, kind", KINDS)
def test_gradients(shape, kind, field, every):
    grids, dt, n_tines = _grids(shape, kind, field)
    out = []
    for g in grids:
        g.forward_checkpointed(13, dt, every)
        w = np.random.default_rng(4).uniform(0.5, 1.0, shape).astype(np.float32)
        dP, _, dperf = g.adjoint(w, n_tines, 0, want_dperf=True)
        out.append((*g.raw_state(), g.omega(), dP, dperf))
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert np.abs(out[0][3]).max() > 0
