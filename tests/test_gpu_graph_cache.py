"""Captured solve loops: more loops than the cache keeps, of one grid shape (one graph a call) and of
several (a graph per shape), without a wait between the calls; a second pass over the same loops
repeats the first one's bits, and the last one matches the FP64 oracle."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, say, to_dev

pytestmark = pytest.mark.gpu

PHASE_TOL = 1e-3   # the parity tests' bar


@pytest.mark.parametrize("shapes", [[(128, 128)], [(128, 128), (256, 128), (128, 128), (128, 256)]])
def test_more_loops_than_the_cache_keeps(shapes):
    from paper_2503_20146_amd import PWF
    import torch
    dev = device()
    rng = np.random.default_rng(len(shapes))
    probs, refs, ys = [], [], []
    for i, (ny, nx) in enumerate(shapes):
        geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx)
        t = S.diffuser(rng, ny, nx)
        refs.append(O.make_problem(t, geo))
        ys.append(S.poisson_intensity(O.physical_model(S.phase_object(rng, ny, nx, 4.0, 2.0), refs[-1])[0], (9, i)))
        probs.append(gpu_problem(geo, t, dev))
    batch, yd = PWF(probs), [to_dev(y, dev) for y in ys]
    counts = range(1, 20)
    passes = []
    for p in range(2):
        say(f"pass {p} over {len(counts)} loops of {len(shapes)} instances")
        passes.append([batch.solve(yd, k)[0] for k in counts])
    torch.cuda.synchronize()
    for a, b in zip(*passes):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    for i, ref in enumerate(refs):
        want, _, _ = O.pwf(ys[i], ref, counts[-1])
        assert np.sqrt(np.mean(np.abs(passes[1][-1][i].cpu().numpy() - want) ** 2)) <= PHASE_TOL
