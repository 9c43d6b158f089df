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


@pytest.mark.parametrize("shape", [(3, 4097, 4099), (5, 3, 1 << 23), (3, 4096, 4096)])
def test_planes_of_2_24_voxels_and_more(shape):
    """Plane strides that 24-bit multiplies do not take: sampled voxels, the
    last ones of rows, planes and grid among them, against the interpolant in
    double."""
    from paper_1907_05709_amd import rfa
    spacing = (0.8e-3, 0.9e-3, 0.7e-3)
    gen = torch.Generator("cuda").manual_seed(5)
    T = 37.0 + 300.0 * torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen)
    v = 6e-3 * (torch.rand((3, *shape), device="cuda", generator=gen) - 0.5)
    g = rfa.Grid(shape, spacing, device=True)
    g.set_tissue(torch.ones(shape, dtype=torch.uint8, device="cuda"), W.standard_tissue())
    g.set_temperature(T)
    out = g.warp(v, 0.7)
    torch.cuda.synchronize()
    rng = np.random.default_rng(6)
    at = np.stack([rng.integers(0, n, 20000) for n in shape])
    ends = np.array([(i, j, k) for i in (0, shape[0] - 1) for j in (0, shape[1] - 1)
                     for k in (0, 1, shape[2] - 2, shape[2] - 1)]).T
    at = torch.from_numpy(np.concatenate([at, ends], axis=1)).cuda()
    base, frac = [], []
    for a in range(3):
        s = at[a].double() + (0.7 / spacing[a]) * v[a][tuple(at)].double()
        s = s.clamp(0.0, shape[a] - 1.0)
        k = s.floor().long().clamp_max(shape[a] - 2)
        base.append(k)
        frac.append(s - k)
    want = torch.zeros_like(frac[0])
    for c in range(8):
        w = torch.ones_like(want)
        for a in range(3):
            w = w * (frac[a] if c >> a & 1 else 1.0 - frac[a])
        want += w * T[tuple(base[a] + (c >> a & 1) for a in range(3))]
    assert (out[tuple(at)].double() - want).abs().max() <= GATE
    g.close()
