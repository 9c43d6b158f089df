"""coverage_loss on a torch that lacks a name it asks about tensors with:
tensor operations take over.  Stand-ins for GPU tensors reach every question
without a GPU."""
from __future__ import annotations

import pytest
import torch

from paper_1907_05709_amd import autograd


class _Names:
    """A module with one name missing."""

    def __init__(self, module, missing):
        self._module, self._missing = module, missing

    def __getattr__(self, name):
        if name == self._missing:
            raise AttributeError(name)
        return getattr(self._module, name)


class _OnGpu(torch.Tensor):
    is_cuda = True


@pytest.mark.parametrize("owner, name", [
    ("torch._C", "_has_storage"), ("torch._C", "_functorch"),
    ("torch._C._functorch", "peek_interpreter_stack"),
    ("torch.autograd.forward_ad", "_current_level"),
    ("torch._C", "_len_torch_dispatch_stack"), ("torch._C", "_len_torch_function_stack")])
def test_a_missing_name_means_tensor_operations(monkeypatch, owner, name):
    om, labels = torch.rand(4, 5, 6), torch.randint(0, 4, (4, 5, 6), dtype=torch.uint8)
    want = autograd._coverage_ops(om, labels, 1e-9, 2, 1, 0.1)
    on_gpu = [t.as_subclass(_OnGpu) for t in (om, labels)]

    class Torch:  # torch as the module under test sees it
        Tensor, nn, strided, jit = _OnGpu, torch.nn, torch.strided, torch.jit
        _C, autograd = torch._C, torch.autograd

    if owner == "torch._C":
        Torch._C = _Names(torch._C, name)
    elif owner == "torch._C._functorch":
        Torch._C = _Names(torch._C, None)
        Torch._C._functorch = _Names(torch._C._functorch, name)
    else:
        Torch.autograd = _Names(torch.autograd, None)
        Torch.autograd.forward_ad = _Names(torch.autograd.forward_ad, name)
    with monkeypatch.context() as m:
        m.setattr(autograd, "torch", Torch)
        with torch._C.DisableTorchFunctionSubclass():
            assert autograd._plain(*on_gpu) is False
    # the loss itself, with what lacks the name answering no
    monkeypatch.setattr(autograd, "_plain", lambda *t: False)
    assert torch.equal(autograd.coverage_loss(om, labels, 1e-9), want)


def test_nothing_missing_means_the_kernels(monkeypatch):
    """The stand-ins reach every question: with all names there the answer is
    yes."""
    om, labels = torch.rand(4, 5, 6), torch.randint(0, 4, (4, 5, 6), dtype=torch.uint8)

    class Torch:
        Tensor, nn, strided, jit = _OnGpu, torch.nn, torch.strided, torch.jit
        _C, autograd = torch._C, torch.autograd

    monkeypatch.setattr(autograd, "torch", Torch)
    with torch._C.DisableTorchFunctionSubclass():
        assert autograd._plain(*(t.as_subclass(_OnGpu) for t in (om, labels))) is True
