"""A solve of 0 iterations of several instances per grid shape, given in mixed order, in a workspace that
an earlier solve has left full: every class clears its own fields, all of them, and psi is exactly 0."""

import dataclasses

import numpy as np
import pytest

import synthetic as S
from gpu_helpers import device, gpu_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [True, False])
def test_zero_iterations_of_several_classes(graphs):
    from paper_2503_20146_amd import PWF, set_graph_mode
    import torch
    dev = device()
    shapes = [(128, 256), (128, 128), (256, 128), (128, 256), (512, 128), (128, 128), (128, 256), (256, 128)]
    rng = np.random.default_rng(3)
    batch = PWF([gpu_problem(dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx), S.diffuser(rng, ny, nx), dev)
                 for ny, nx in shapes])
    y = [1 + 0.2 * torch.rand(s, device=dev) for s in shapes]
    say(f"0 iterations of {shapes}, graphs {graphs}")
    set_graph_mode(graphs)
    try:
        assert all(float(o.abs().max()) > 0 for o in batch.solve(y, 3)[0])
        assert all(bool((o == 0).all()) for o in batch.solve(y, 0)[0])
    finally:
        set_graph_mode(True)
