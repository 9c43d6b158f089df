"""What rfa_kernel_stats counts when launches take two steps: every launch of
an automatic plan, of calls of one step among them; only the launches of two
where depth 2 was asked for."""
from __future__ import annotations

import pytest

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("diag", [False, True])
@pytest.mark.parametrize("period", [1, 16])
@pytest.mark.parametrize("kw, launches, steps", [
    ({}, lambda n: n // 2 + n % 2, lambda n: n),
    (dict(depth=2), lambda n: n // 2, lambda n: n // 2 * 2),
    (dict(depth=1), lambda n: n, lambda n: n),
])
def test_launches_and_voxel_steps(kw, launches, steps, period, diag):
    case = W.case_straight(n=32, n_steps=20, seed=2007)
    g = rfa.Grid(case.shape, case.spacing, time_kernels=period, **kw)
    g.load_case(case)
    for n in (1, 2, 5, 150, 2049):
        g.step(n, case.dt, diag=diag)
        ms, count, voxel_steps = g.kernel_stats()
        # a call runs in stretches of 1024 steps, each of whole launches
        assert (count, voxel_steps) == (launches(n), steps(n) * case.n_voxels), n
        assert (ms > 0.0) == (count > 0), n
    g.step(1, case.dt, diag=diag)
    g.step(1, case.dt, diag=diag)
    assert g.kernel_stats()[1] == 2 * launches(1)
    g.close()
