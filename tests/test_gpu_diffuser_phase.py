"""Backward factor of the diffuser estimate, one Fourier mode at a time.

With no source blur and eps = 0 the estimate of a reference 1 + 0.9 cos(k r) is the square root
propagated back over L2.  The coefficient of its mode k, divided by the one that the same reference gives at
L2 = 0 (which takes out what the transforms do to this mode), is the library's conj Q_L2(k):
rounding of the pixels averages out over the projection.  The factor must be cos and sin of ONE phase, formed in
FP64 and rounded to FP32.  Against the FP64 cosine and sine of that rounded phase, FP32 results
within an ulp of 2^-24 are off by an RMS of at most 2^-24 / sqrt(3) in each part, sqrt(2) of that
together: 4.9e-8.  (A product of two factors with a rounded phase each is off by 8e-8.)
"""

import dataclasses

import numpy as np
import pytest

import synthetic as S
from gpu_helpers import device, gpu_problem, say, to_dev

pytestmark = pytest.mark.gpu

TOL = 2.0 ** -24 * np.sqrt(2.0 / 3.0)


@pytest.mark.parametrize("ny,nx,wavelength_m", [(128, 128, 0.05e-9), (128, 256, 0.05e-9), (128, 128, 5e-8)])
def test_backward_factor_has_one_rounded_phase(ny, nx, wavelength_m):
    from paper_2503_20146_amd import diffuser_from_reference
    dev = device()
    geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx, sigma_x_px=0.0, sigma_y_px=0.0,
                              wavelength_m=wavelength_m)
    p = gpu_problem(geo, np.ones((ny, nx)), dev)
    p0 = gpu_problem(dataclasses.replace(geo, z2_m=0.0), np.ones((ny, nx)), dev)
    rng = np.random.default_rng(ny + nx)
    say(f"diffuser phase {ny} x {nx}, wavelength {wavelength_m}")
    lp = wavelength_m / geo.pixel_m
    err = []
    for _ in range(300):
        kx, ky = int(rng.integers(1, nx // 2)), int(rng.integers(1, ny // 2)) * int(rng.choice((-1, 1)))
        arg = 2 * np.pi * ((kx * np.arange(nx)[None, :] / nx + ky * np.arange(ny)[:, None] / ny) % 1.0)
        ref = (1 + 0.9 * np.cos(arg)).astype(np.float32)
        mode = np.exp(-1j * arg)
        c, c0 = (np.sum(diffuser_from_reference(q, to_dev(ref, dev), 0.0).cpu().numpy().astype(np.complex128) * mode)
                 for q in (p, p0))
        r2 = (kx / nx) ** 2 + (ky / ny) ** 2
        rev = -geo.z2_m * wavelength_m / (2 * geo.pixel_m ** 2) * r2 * 2 / (1 + np.sqrt(1 - lp * lp * r2))
        phase = float(np.float32(2 * np.pi * (rev - np.rint(rev))))
        err.append(abs(c / c0 - np.exp(-1j * phase)))
    rms = float(np.sqrt(np.mean(np.square(err))))
    assert rms <= TOL
