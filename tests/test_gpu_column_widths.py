"""Column tile widths chosen by the size of the batch: the largest and smallest batches on either
side of each limit, every instance the same, against the FP64 oracle (psi and the loss, whose
partials are counted per tile) and against one instance on its own."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, say, to_dev

pytestmark = pytest.mark.gpu

PHASE_TOL = LOSS_TOL = 1e-3   # the parity tests' bar


@pytest.mark.parametrize("ny,nx,count", [(1024, 128, 80), (1024, 128, 81), (2048, 128, 63), (2048, 128, 64)])
def test_widths_around_the_limits(ny, nx, count):
    from paper_2503_20146_amd import PWF
    import torch
    dev = device()
    geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx)
    rng = np.random.default_rng(count)
    t = S.diffuser(rng, ny, nx)
    prob = O.make_problem(t, geo)
    y = S.poisson_intensity(O.physical_model(S.phase_object(rng, ny, nx, 4.0, 2.0), prob)[0], (21, count))
    p, yd = gpu_problem(geo, t, dev), to_dev(y, dev)
    say(f"{count} x {ny} x {nx}")
    out, hist = PWF([p] * count).solve([yd] * count, 4)
    want, losses, _ = O.pwf(y, prob, 4)
    assert all(torch.equal(out[0], o) for o in out)
    assert np.sqrt(np.mean(np.abs(out[0].cpu().numpy() - want) ** 2)) <= PHASE_TOL
    assert np.allclose(hist[count - 1].cpu().numpy(), losses, rtol=LOSS_TOL)
    one, _ = PWF([p]).solve([yd], 4)
    assert float((out[0] - one[0]).abs().square().mean().sqrt()) <= PHASE_TOL
