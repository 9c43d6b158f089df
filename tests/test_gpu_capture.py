"""Library calls captured in a HIP graph: replays read and write the grid's
state as it is at the replay, whatever steps were taken in between."""
from __future__ import annotations

import dataclasses

import pytest
import torch

from paper_1907_05709_amd import rfa
from paper_1907_05709_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(shape, coupled=False):
    return dataclasses.replace(W.random_tissue_case(61, shape=shape, n_classes=4, n_tines=2),
                               perfusion_decay=coupled)


def _grid(case, stream, **kw):
    g = rfa.Grid(case.shape, case.spacing, device=True, stream=stream.cuda_stream, A=6.0e8,
                 Ea=5.0e4, **kw)
    g.load_case(case)
    torch.cuda.synchronize()
    return g


def _omega(g):
    """The damage integral, waited for: the read is only enqueued on the
    grid's stream, which torch's own is not ordered with."""
    torch.cuda.synchronize()
    om = g.omega()
    torch.cuda.synchronize()
    return om


def _captured(stream, call):
    """The graph of call() on the stream and what call() returned."""
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = call()
    torch.cuda.synchronize()
    return graph, out


def test_captured_damage_follows_coupled_steps():
    """Damage-coupled grids step between two damage images; a captured
    rfa_damage_noalloc reads the grid's own, after any number of steps."""
    case = _case((26, 33, 40), coupled=True)
    stream = torch.cuda.Stream()
    g = _grid(case, stream)
    dt = 0.9 * min(case.dt, g.dt_max())
    assert g.plan()["depth"] == 2
    g.damage_noalloc(want_dead=False)  # looks the scratch up before the capture
    graph, (mask, omega, _) = _captured(stream, lambda: g.damage_noalloc(want_dead=False))
    last = None
    for n in (2, 2, 3, 4, 6, 1, 2):
        g.step(n, dt, diag=False)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = g.damage()
        torch.cuda.synchronize()
        assert torch.equal(omega, want[1]) and torch.equal(mask, want[0]), n
        assert last is None or not torch.equal(omega, last), n
        last = omega.clone()
    g.close()


@pytest.mark.parametrize("coupled", [False, True])
def test_steps_allocate_nothing(coupled):
    """A program that has taken single steps only may capture a longer call:
    what two steps a launch need is there since the tissue was set."""
    case = _case((26, 33, 40), coupled)
    stream = torch.cuda.Stream()
    g, ref = _grid(case, stream), _grid(case, stream, kernel=1)
    dt = 0.9 * min(case.dt, g.dt_max())
    assert g.plan()["depth"] == 2
    for x in (g, ref):
        x.step(1, dt, diag=False)
    torch.cuda.synchronize()
    graph, _ = _captured(stream, lambda: g.step(4, dt, diag=False))
    for _ in range(3):
        graph.replay()
        ref.step(4, dt, diag=False)
        torch.cuda.synchronize()
        for a, b in zip(g.raw_state(), ref.raw_state()):
            assert torch.equal(a, b)
        assert torch.equal(_omega(g), _omega(ref))
    for x in (g, ref):
        x.close()


@pytest.mark.parametrize("coupled", [False, True])
@pytest.mark.parametrize("n", [2, 4, 6, 10])
def test_captured_steps_advance_at_every_replay(n, coupled):
    case = _case((20, 31, 44), coupled)
    stream = torch.cuda.Stream()
    g, ref = _grid(case, stream), _grid(case, stream, kernel=1)
    dt = 0.9 * min(case.dt, g.dt_max())
    assert g.plan()["depth"] == 2
    for x in (g, ref):
        x.step(2, dt, diag=False)
    torch.cuda.synchronize()
    graph, _ = _captured(stream, lambda: g.step(n, dt, diag=False))
    for k in (3, 2):
        for _ in range(k):
            graph.replay()
            ref.step(n, dt, diag=False)
        torch.cuda.synchronize()
        for a, b in zip(g.raw_state(), ref.raw_state()):
            assert torch.equal(a, b)
        # the grid's own steps, of any even number, in between
        for x in (g, ref):
            x.step(6, dt, diag=False)
        assert torch.equal(_omega(g), _omega(ref))
    for x in (g, ref):
        x.close()


def test_captured_view_follows_even_steps():
    """A captured view shows the state after any even number of steps, taken
    by the grid or by a batch."""
    case = _case((20, 31, 44))
    stream = torch.cuda.Stream()
    g = _grid(case, stream)
    dt = 0.9 * min(case.dt, g.dt_max())
    assert g.plan()["depth"] == 2
    v = 2e-3 * torch.rand((3, *case.shape), device="cuda",
                          generator=torch.Generator("cuda").manual_seed(3))
    b = rfa.Batch([g], [dt])
    b.step(2)
    g.step(2, dt, diag=False)
    out = torch.empty(case.shape, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    graph, _ = _captured(stream, lambda: g.warp(v, 0.7, out=out))
    for n in (2, 2, 4, 6, 10):
        for step in (lambda: g.step(n, dt, diag=False), lambda: b.step(n)):
            step()
            torch.cuda.synchronize()
            graph.replay()
            want = g.warp(v, 0.7)
            torch.cuda.synchronize()
            assert torch.equal(out, want), n
    b.close()
    g.close()
