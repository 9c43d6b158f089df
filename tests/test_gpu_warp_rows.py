"""The breathing view at the edges of its launch: rows of fewer than four
voxels, rows that four does not divide, planes of fewer threads than XCDs'
eighths, and displacements that are not finite.

Tolerance (K), below 1024 degC: the dropped lo words (ulp(hi) / 2 of an
excess below 1024 K, 3.1e-5), the output rounding (3.1e-5) and the lerps'
roundings on corner excesses of at most 600 K (~4 eps 600 = 1.5e-4 at the
very most, weighted by fractions; 2.4e-5 for one difference of 400 K):
1e-4, as for the ordinary shapes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle.warp import warp as warp_oracle
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu
GATE = 1e-4


def _grid(shape, spacing, T, device=False):
    from paper_1907_05709_amd import rfa
    case = W.random_tissue_case(6100, shape=shape, n_classes=3, n_tines=1, n_steps=5)
    g = rfa.Grid(shape, spacing, device=device)
    on = (lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()) if device else (lambda a: a)
    g.set_tissue(on(case.labels), case.tissue)
    g.set_temperature(on(T))
    return g


@pytest.mark.parametrize("shape", [(4, 3, 3), (3, 17, 3), (3, 3, 4), (9, 4, 5), (7, 11, 6),
                                   (6, 9, 7), (5, 3, 1027), (3, 300, 9)])
@pytest.mark.parametrize("two", [False, True])
def test_rows_of_any_length(shape, two):
    spacing = (0.8e-3, 0.9e-3, 0.7e-3)
    T = W.hot_field(shape, spacing, peak_c=600.0, sigma_m=4e-3, seed=41 + shape[2])
    v = W.breathing_field(shape, spacing, amplitude_m=2e-3, seed=42)
    w = W.breathing_field(shape, spacing, amplitude_m=3e-3, seed=43)
    g = _grid(shape, spacing, T)
    if two:
        out = g.warp(v, 0.6, v2=w, beta2=0.4)
        ref = warp_oracle(T, 0.6 * v.astype(np.float64) + 0.4 * w.astype(np.float64), spacing, 1.0)
    else:
        out = g.warp(v, -0.8)
        ref = warp_oracle(T, v, spacing, -0.8)
    err = np.abs(out.astype(np.float64) - ref).max()
    print(shape, two, "max err", err)
    assert err <= GATE
    g.close()


def test_displacements_that_are_not_finite():
    """On the device, where the field is not checked, +-inf and values beyond
    any voxel index sample the walls, a NaN the lower wall; neighbouring
    voxels are untouched."""
    shape, spacing = (6, 7, 13), (1e-3,) * 3
    T = W.hot_field(shape, spacing, peak_c=600.0, sigma_m=4e-3, seed=44)
    v = W.breathing_field(shape, spacing, amplitude_m=2e-3, seed=45)
    far = v.copy()
    for k, (bad, wall) in enumerate([(np.inf, 1e3), (-np.inf, -1e3), (np.nan, -1e3),
                                     (3e38, 1e3), (-3e38, -1e3)]):
        for a in range(3):
            at = (a, 1 + k % 4, 2 + a, 3 + 2 * k)
            v[at], far[at] = bad, wall
    g = _grid(shape, spacing, T, device=True)
    out = g.warp(torch.from_numpy(v).cuda(), 1.0).cpu().numpy()
    ref = warp_oracle(T, far, spacing, 1.0)
    assert np.isfinite(out).all()
    assert np.abs(out.astype(np.float64) - ref).max() <= GATE
    assert np.array_equal(out, g.warp(torch.from_numpy(far).cuda(), 1.0).cpu().numpy())
    g.close()
