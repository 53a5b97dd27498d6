"""The cache of captured solves never makes a call wait for the GPU, and a solve can be part of a
caller's own graph.

* With the GPU held by a long kernel, calls that find the cache full of solves in flight (more solves
  than it keeps; more grid shapes in one batch than solves; batches of several shapes in turn) return
  before that kernel ends, with the results of the same calls made one at a time.
* Solves of one and of several grid shapes captured into a caller's graph, as a first and as a later
  call, with the library's own graphs on and off, and a batch whose descriptors are staged outside a
  capture: every replay gives the bits of the eager call, with other solves between the replays.
"""

import dataclasses
import itertools

import numpy as np
import pytest

import synthetic as S
from gpu_helpers import device, gpu_problem, say

pytestmark = pytest.mark.gpu


def make_batch(shapes, seed, dev):
    from paper_2503_20146_amd import PWF
    import torch
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=dev).manual_seed(seed)
    probs = [gpu_problem(dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx), S.diffuser(rng, ny, nx), dev)
             for ny, nx in shapes]
    return PWF(probs), [1 + 0.2 * torch.rand(s, device=dev, generator=g) for s in shapes]


def hold_gpu(seconds):
    """A kernel that keeps the GPU busy for about `seconds`, and an event behind it."""
    import torch
    e0, e1, behind = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    e0.record()
    torch.cuda._sleep(10_000_000)
    e1.record()
    e1.synchronize()
    torch.cuda._sleep(int(10_000_000 * seconds * 1e3 / e0.elapsed_time(e1)))
    behind.record()
    return behind


SHAPES = list(itertools.product((128, 256, 512, 1024), repeat=2)) + [(128, 2048), (2048, 128)]


@pytest.mark.parametrize("batches", [[[(128, 128)]] * 18, [SHAPES],
                                     [[(128, 128), (128, 256), (256, 128)]] * 6 + [[(256, 256)]] * 11])
def test_calls_return_while_the_gpu_is_busy(batches):
    import torch
    dev = device()
    made = [make_batch(b, i, dev) for i, b in enumerate(batches)]
    say(f"{len(made)} solves of {[len(b) for b in batches]} grid shapes")
    want = []
    for batch, y in made:   # (also first passes of every kernel)
        want.append(batch.solve(y, 2)[0])
        torch.cuda.synchronize()
    behind = hold_gpu(1.0)
    got = [batch.solve(y, 2)[0] for batch, y in made] + [batch.solve(y, 2)[0] for batch, y in made]
    returned_early = not behind.query()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for w, g in zip(want + want, got) for a, b in zip(w, g))
    assert returned_early


@pytest.mark.parametrize("own_graphs", [True, False])
@pytest.mark.parametrize("warm", [True, False])
@pytest.mark.parametrize("shapes", [[(128, 256)], [(128, 128), (256, 128), (128, 128)]])
def test_solve_in_a_callers_graph(shapes, warm, own_graphs):
    from paper_2503_20146_amd import set_graph_mode
    import torch
    dev = device()
    batch, y = make_batch(shapes, 5, dev)
    other, y2 = make_batch(shapes, 6, dev)
    say(f"capture of a solve of {shapes}, warm {warm}, own graphs {own_graphs}")
    set_graph_mode(own_graphs)
    try:
        other.solve(y2, 3)
        if warm:
            batch.solve(y, 3)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out, hist = batch.solve(y, 3)
        want, want_hist = batch.solve(y, 3)
        for _ in range(4):
            for o in out:
                o.fill_(float("nan"))
            other.solve(y2, 3)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(out, want)) and torch.equal(hist, want_hist)
    finally:
        set_graph_mode(True)


def test_large_batch_in_a_callers_graph():
    """More instances than a set-up launch or four carry: the graph holds its own descriptors."""
    import torch
    dev = device()
    n = 45
    batch, y = make_batch([(128, 128)] * n, 7, dev)
    other, y2 = make_batch([(128, 256)] * n, 8, dev)
    say(f"capture of a solve and a forward call of {n} instances")
    other.solve(y2, 2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out, hist = batch.solve(y, 2)
        f = batch.forward(out)
    want, want_hist = batch.solve(y, 2)
    want_f = batch.forward(want)
    for _ in range(6):
        for o in out + f:
            o.fill_(float("nan"))
        for _ in range(5):   # (every slot of the staging ring is used by other calls)
            other.forward(other.solve(y2, 1)[0])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out + f, want + want_f)) and torch.equal(hist, want_hist)


def test_large_noalloc_batch_in_a_callers_graph():
    import torch
    dev = device()
    n = 45
    batch, y = make_batch([(128, 128)] * n, 9, dev)
    other, y2 = make_batch([(128, 128)] * n, 10, dev)
    psi = [0.1 * torch.randn(128, 128, dtype=torch.complex64, device=dev) for _ in range(n)]
    say(f"capture of the loss and gradient of {n} instances without a workspace")
    want_loss, want = batch.loss_grad_noalloc(psi, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loss, grad = batch.loss_grad_noalloc(psi, y)
    for _ in range(4):
        for g in grad:
            g.fill_(float("nan"))
        other.loss_grad_noalloc(psi, y2)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(grad, want)) and torch.equal(loss, want_loss)
