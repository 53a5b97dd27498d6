"""Speckle autocorrelations and the diffuser estimate where their kernels change: images that
the 64-column tiles do not divide, one-wrap margins (images barely wider than the shifts), fewer
shifts than lanes, tall and short tiles, and the sweeps of the diffuser estimate on split and
unsplit column transforms and non-square grids; against the FP64 oracle."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,shift", [(33, 33, 32), (64, 64, 32), (47, 200, 32), (130, 65, 7), (5, 3, 2), (1, 9, 0),
                                         (1000, 1537, 32)])
def test_g2_tiles(ny, nx, shift):
    """FP64 products and sums on both sides: only the order of the sums differs (1e-12)."""
    from paper_2503_20146_amd import speckle_g2
    dev = device()
    rng = np.random.default_rng(ny + nx)
    ref = rng.gamma(2.0, 0.5, (ny, nx)).astype(np.float32)
    say(f"speckle g2 {ny} x {nx}, {shift} shifts")
    gx, gy = speckle_g2(to_dev(ref, dev), shift)
    rx, ry = O.speckle_g2(ref.astype(np.float64), shift)
    assert len(gx) == len(gy) == shift + 1
    assert np.max(np.abs(np.array(gx) / rx - 1)) <= 1e-12
    assert np.max(np.abs(np.array(gy) / ry - 1)) <= 1e-12


@pytest.mark.parametrize("ny,nx", [(128, 256), (256, 128), (512, 128), (256, 2048)])
def test_diffuser_shapes(ny, nx):
    """Relative L2 1e-4, the bound of test_gpu_calibration (the square root amplifies the
    rounding of intensities near zero)."""
    from paper_2503_20146_amd import diffuser_from_reference
    dev = device()
    geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx, sigma_x_px=1.3, sigma_y_px=0.9)
    rng = np.random.default_rng(nx)
    t = S.diffuser(rng, ny, nx)
    prob = O.make_problem(t, geo)
    f, _, _ = O.physical_model(np.zeros((ny, nx), np.complex128), prob)
    ref = S.poisson_intensity(f, (1, nx))
    say(f"diffuser estimate {ny} x {nx}")
    got = diffuser_from_reference(gpu_problem(geo, t, dev), to_dev(ref, dev), 1e-2).cpu().numpy()
    assert rel(got, O.diffuser_from_reference(ref.astype(np.float64), prob, 1e-2)) <= 1e-4
