"""A field's forward model has the same bits whatever else is in the call: alone, in batches on both
sides of 1 M pixels of small grids, and beside grids of other sizes."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, rel, say, to_dev

pytestmark = pytest.mark.gpu

FWD_TOL = 1e-5   # the parity tests' bar


def scene(ny, nx, dev):
    geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx)
    rng = np.random.default_rng(ny + 2 * nx)
    psi, t = S.phase_object(rng, ny, nx, 4.0, 2.0).astype(np.complex64), S.diffuser(rng, ny, nx)
    f_ref, _, _ = O.physical_model(psi.astype(np.complex128), O.make_problem(t, geo))
    return gpu_problem(geo, t, dev), to_dev(psi, dev), f_ref


@pytest.mark.parametrize("ny,nx,counts", [(128, 128, (64, 65)), (256, 256, (16, 17)), (128, 256, (32, 33))])
def test_forward_has_the_same_bits_in_every_batch(ny, nx, counts):
    from paper_2503_20146_amd import PWF
    import torch
    dev = device()
    p, psi, f_ref = scene(ny, nx, dev)
    q, other, _ = scene(512, 512, dev)
    y = torch.ones(ny, nx, device=dev)
    say(f"forward of {ny} x {nx} alone and in batches of {counts}")
    one, err = PWF([p]).forward([psi])[0], PWF([p]).rmse_image([psi], [y], [1.0])[0]
    assert rel(one.cpu().numpy(), f_ref) <= FWD_TOL
    for n in counts:
        batch = PWF([p] * n)
        assert all(torch.equal(one, f) for f in batch.forward([psi] * n))
        assert all(torch.equal(err, r) for r in batch.rmse_image([psi] * n, [y] * n, [1.0] * n))
    assert torch.equal(one, PWF([q, p]).forward([other, psi])[1])
