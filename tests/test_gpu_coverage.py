"""The coverage loss through the library's kernels against the same loss as
tensor operations in double.

Tolerances: the sums are over at most 2^18 terms of at most 1 in double, in
another order (2^18 eps = 6e-11 at the very most; pairwise sums are near
1e-15): 1e-12 relative.  Gradients are the float32 of a double formed from
the same factors: half an ulp on either side, 1.2e-7 relative."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_1907_05709_amd import autograd

pytestmark = pytest.mark.gpu
VOX = 0.4e-9


def _inputs(shape, seed=7):
    rng = np.random.default_rng(seed)
    om = np.exp(rng.uniform(-14, 14, size=shape)).astype(np.float32)
    special = np.array([0.0, -1.0, np.nan, np.inf, 1e-38, 1e-12, 1.0, 3e38, -np.inf], np.float32)
    flat = om.reshape(-1)
    flat[:: max(1, flat.size // special.size)][: special.size] = special[: flat[
        :: max(1, flat.size // special.size)].size]
    labels = rng.integers(0, 5, size=shape).astype(np.uint8)
    return torch.from_numpy(om).cuda(), torch.from_numpy(labels).cuda()


def _both(om, labels, **kw):
    out = []
    for f in (autograd.coverage_loss,
              lambda o, l, v, tumour=2, liver=1, healthy_weight=0.1:
              autograd._coverage_ops(o, l, v, tumour, liver, healthy_weight)):
        o = om.detach().clone().requires_grad_(True)
        loss = f(o, labels, VOX, **kw)
        (3.0 * loss).backward()
        out.append((loss.detach(), o.grad))
    return out


def _same(a, b):
    assert a[0].dtype == b[0].dtype == torch.float64 and a[0].shape == b[0].shape
    assert torch.allclose(a[0], b[0], rtol=1e-12, atol=1e-300)
    assert a[1].dtype == torch.float32
    assert torch.allclose(a[1], b[1], rtol=1.2e-7, atol=1e-44)


@pytest.mark.parametrize("shape", [(1,), (3,), (4, 1, 1), (7, 5, 3), (63, 4, 4), (37, 41, 43),
                                   (64, 64, 64)])
@pytest.mark.parametrize("kw", [{}, dict(tumour=3, liver=3), dict(tumour=200, healthy_weight=2)])
def test_loss_and_gradient_equal_tensor_operations(shape, kw):
    om, labels = _inputs(shape)
    fast, ops = _both(om, labels, **kw)
    _same(fast, ops)
    with torch.no_grad():
        assert torch.equal(autograd.coverage_loss(om, labels, VOX, **kw), fast[0])


def test_views_layouts_and_types():
    """Tensors that start anywhere in their storage, strided ones and other
    types: the same loss whichever path takes them."""
    om, labels = _inputs((9, 11, 13))
    ref = autograd._coverage_ops(om, labels, VOX, 2, 1, 0.1)
    at = torch.empty(om.numel() + 1, device="cuda")[1:].view(om.shape).copy_(om)
    lt = torch.empty(om.numel() + 3, dtype=torch.uint8, device="cuda")[3:].view(om.shape)
    lt.copy_(labels)
    strided = om.transpose(0, 2).contiguous().transpose(0, 2)
    for o, l in ((at, lt), (strided, labels), (om, labels.long()), (om.double(), labels),
                 (om.cpu(), labels.cpu()), (om[::2], labels[::2])):
        want = ref if o.shape == om.shape else autograd._coverage_ops(o, l, VOX, 2, 1, 0.1)
        assert torch.allclose(autograd.coverage_loss(o, l, VOX).cpu(), want.cpu(), rtol=1e-12)
    _same(*_both(at, lt))


def test_inputs_may_change_before_the_gradient():
    om, labels = _inputs((8, 8, 8))
    _, want = _both(om, labels)[1]
    leaf = om.clone().requires_grad_(True)
    o = leaf * 1.0
    loss = autograd.coverage_loss(o, labels, VOX)
    with torch.no_grad():
        o.zero_()
        labels.zero_()
    (3.0 * loss).backward()
    assert torch.allclose(leaf.grad, want, rtol=1.2e-7, atol=1e-44)


def test_second_derivatives_transforms_and_hooks():
    om, labels = _inputs((5, 6, 7))
    om = torch.nan_to_num(om, nan=0.5, posinf=2.0, neginf=0.0).clamp(1e-3, 1e3)
    second = []
    for f in (lambda o: autograd.coverage_loss(o, labels, VOX),
              lambda o: autograd._coverage_ops(o, labels, VOX, 2, 1, 0.1)):
        o = om.clone().requires_grad_(True)
        (g,) = torch.autograd.grad(f(o), o, create_graph=True)
        (h,) = torch.autograd.grad((g * g.detach()).sum(), o)
        second.append((g.detach(), h))
    scale = [t.abs().max() for t in second[1]]
    assert (second[0][0] - second[1][0]).abs().max() <= 1e-6 * scale[0]
    assert (second[0][1] - second[1][1]).abs().max() <= 1e-5 * scale[1]
    # several upstream gradients at once
    o = om.clone().requires_grad_(True)
    up = torch.tensor([1.0, -2.0], dtype=torch.float64, device="cuda")
    (b,) = torch.autograd.grad(autograd.coverage_loss(o, labels, VOX), o, up, is_grads_batched=True)
    assert torch.allclose(b[1], -2.0 * b[0]) and torch.allclose(b[0], second[1][0], rtol=1e-6)
    # functional transforms and forward mode
    f = lambda x: autograd.coverage_loss(x, labels, VOX)  # noqa: E731
    assert torch.allclose(torch.func.grad(f)(om), second[1][0], rtol=1e-6)
    v = torch.vmap(f)(torch.stack([om, 2 * om]))
    assert torch.allclose(v, torch.stack([f(om), f(2 * om)]), rtol=1e-12)
    _, t = torch.func.jvp(f, (om,), (torch.ones_like(om),))
    assert torch.allclose(t, second[1][0].double().sum(), rtol=1e-5)
    # kept tensors pass through the caller's hooks
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda x: seen.append(x) or x.cpu(),
                                                  lambda x: x.cuda()):
        o = om.clone().requires_grad_(True)
        loss = autograd.coverage_loss(o, labels, VOX)
    loss.backward()
    assert seen and torch.allclose(o.grad, second[1][0], rtol=1e-6)


@pytest.mark.parametrize("how", ["script", "compile", "trace", "fx", "make_fx"])
def test_compilers_and_tracers_take_the_tensor_operations(how):
    om, labels = _inputs((4, 5, 6))
    f = lambda o: autograd.coverage_loss(o, labels, VOX)  # noqa: E731
    if how == "script":
        g = torch.jit.script(autograd.coverage_loss)
        got = g(om, labels, VOX)
    elif how == "compile":
        got = torch.compile(autograd.coverage_loss, backend="eager", fullgraph=True)(om, labels, VOX)
    elif how == "trace":
        got = torch.jit.trace(f, om)(om)
    elif how == "fx":
        got = torch.fx.symbolic_trace(f)(om)
    else:
        from torch.fx.experimental.proxy_tensor import make_fx
        got = make_fx(f)(om)(om)
    assert torch.allclose(got, f(om), rtol=1e-12)


@pytest.mark.parametrize("upstream, weight", [(np.inf, 0.1), (-np.inf, 0.0), (np.nan, 0.1),
                                              (1.0, np.inf), (1.0, np.nan)])
def test_gradients_that_are_not_finite(upstream, weight):
    """A factor that is not finite shows where it does in the tensor
    operations: on every voxel with damage, whatever its class."""
    om, labels = _inputs((7, 5, 3))
    om = torch.nan_to_num(om, nan=0.5, posinf=2.0, neginf=0.0).clamp_max(1e3)
    grads = []
    for f in (lambda o: autograd.coverage_loss(o, labels, VOX, healthy_weight=weight),
              lambda o: autograd._coverage_ops(o, labels, VOX, 2, 1, weight)):
        o = om.clone().requires_grad_(True)
        f(o).backward(torch.tensor(upstream, dtype=torch.float64, device="cuda"))
        grads.append(o.grad)
    a, b = grads
    assert torch.equal(a.isnan(), b.isnan()) and bool(b.isnan().any())
    assert torch.equal(a.isinf(), b.isinf())
    finite = b.isfinite()
    assert torch.allclose(a[finite], b[finite], rtol=1.2e-7, atol=1e-44)
