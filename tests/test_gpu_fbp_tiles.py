"""Filtered back-projection over the workgroup shapes its dispatch chooses from (8, 4, 2 or 1
slices of 32 x 32, 16 x 32 or 16 x 16 voxels) and over the padded lengths of the ramp filter,
with odd detector widths, odd angle counts and volume sides that the tiles do not divide,
against the FP64 oracle: FP32 filtering and sums, relative L2 1e-5 per slice (the bound of
test_gpu_fbp)."""

import numpy as np
import pytest

import oracle as O
from gpu_helpers import device, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,P,n_out", [
    (512, 32, 21, 512),     # 8 slices, 2 x 2 voxels
    (301, 32, 64, 416),     # 4 slices, 2 x 2
    (1000, 32, 67, 272),    # 4 slices, 1 x 2, a partial z tile; n_pad 2048
    (129, 32, 13, 160),     # 2 slices, 1 x 2
    (64, 64, 5, 48),        # 1 slice, 1 voxel; n_pad 128
    (255, 32, 3, 16),       # the smallest volume
])
def test_fbp_tiles(nx, ny, P, n_out):
    from paper_2503_20146_amd import fbp
    dev = device()
    rng = np.random.default_rng(nx + P)
    angles = np.pi * (np.arange(P) + 0.25) / P
    u = np.arange(nx) + 0.5 - nx / 2.0
    c = rng.uniform(-0.3, 0.3, (6, 2)) * nx
    w = rng.uniform(0.02, 0.1, 6) * nx
    amp = rng.uniform(0.5, 1.5, (6, ny)) * np.exp(1j * rng.uniform(0, 6, (6, ny)))
    sino = np.zeros((P, ny, nx), np.complex64)
    for j, th in enumerate(angles):
        uc = c[:, 0] * np.cos(th) - c[:, 1] * np.sin(th)
        sino[j] = amp.T @ np.exp(-0.5 * ((u[None] - uc[:, None]) / w[:, None]) ** 2)
    say(f"fbp tiles {P} x {ny} x {nx} -> {n_out}^2")
    vol = fbp([to_dev(s, dev) for s in sino], angles, n_out).cpu().numpy()
    for y in (0, 7, ny - 1):
        ref = O.backproject(O.fbp_filter(sino[:, y].astype(np.complex128)), angles, n_out)
        assert rel(vol[y], ref) <= 1e-5
