"""Column tile widths chosen by the size of the batch round as any other: on both sides of each limit,
psi and the loss history of an instance have the bits that they have alone, for one and for several
grid shapes of a batch, and with the other width set by hand (S5's loss partials keep their width)."""

import dataclasses

import numpy as np
import pytest

import synthetic as S
from gpu_helpers import device, gpu_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,count", [(1024, 128, 80), (1024, 128, 81), (2048, 128, 63), (2048, 128, 64)])
def test_an_instance_has_the_same_bits_in_every_batch(ny, nx, count):
    from paper_2503_20146_amd import PWF, set_column_tile
    import torch
    dev = device()
    rng = np.random.default_rng(count)
    p = gpu_problem(dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx), S.diffuser(rng, ny, nx), dev)
    q = gpu_problem(S.config_geometry(0), S.diffuser(rng, 128, 128), dev)
    y, yq = 1 + 0.2 * torch.rand(ny, nx, device=dev), 1 + 0.2 * torch.rand(128, 128, device=dev)
    say(f"{count} x {ny} x {nx}, alone and beside another grid")
    one, hist1 = PWF([p]).solve([y], 4)
    for batch, ys in ((PWF([p] * count), [y] * count), (PWF([q] + [p] * count), [yq] + [y] * count)):
        out, hist = batch.solve(ys, 4)
        assert all(torch.equal(o, one[0]) for o in out[-count:])
        assert all(torch.equal(h, hist1[0]) for h in hist[-count:])
    try:
        for width in (8, 16):
            for sweep in (1, 3, 7, 9, 11):
                set_column_tile(ny, width, sweep)
            out, hist = PWF([p]).solve([y], 4)
            assert torch.equal(out[0], one[0]) and torch.equal(hist[0], hist1[0])
    finally:
        set_column_tile(ny, 0)
