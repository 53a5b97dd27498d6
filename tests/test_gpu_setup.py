"""Set-up of a call at the batch sizes where its route changes (descriptors as kernel arguments in
one launch, in several, or through the staging buffer), and the joint diffuser step with whole
groups of eight instances and a remainder, against the FP64 oracle."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, rel, say, to_dev

pytestmark = pytest.mark.gpu

FWD_TOL, GRAD_TOL, PHASE_TOL = 1e-5, 1e-4, 1e-3   # the bars of the parity tests


def scenes(n, seed):
    """n objects behind two diffusers, sides 128 (so that a batch of 41 stays small)."""
    geo = dataclasses.replace(S.config_geometry(0), ny=128, nx=128)
    rng = np.random.default_rng(seed)
    t = [S.diffuser(rng, 128, 128) for _ in range(2)]
    probs = [O.make_problem(x, geo) for x in t]
    psi = [S.phase_object(rng, 128, 128, 4.0, 2.0) for _ in range(n)]
    f = [O.physical_model(p, probs[i % 2])[0] for i, p in enumerate(psi)]
    return geo, t, probs, psi, f


@pytest.mark.parametrize("n", [1, 10, 11, 40, 41])
def test_batch_sizes_of_the_setup(n):
    from paper_2503_20146_amd import PWF
    dev = device()
    geo, t, probs, psi, f = scenes(n, n)
    td = [gpu_problem(geo, x, dev) for x in t]
    batch = PWF([td[i % 2] for i in range(n)])
    say(f"set-up of {n} instances")
    half = [(0.5 * p).astype(np.complex64) for p in psi]
    y = [S.poisson_intensity(x, (3, i)) for i, x in enumerate(f)]
    pd, yd = [to_dev(h, dev) for h in half], [to_dev(x, dev) for x in y]
    out = batch.forward(pd)
    loss, g, _ = batch.gradient(pd, yd)
    for i in {0, n // 2, n - 1}:
        h = half[i].astype(np.complex128)
        assert rel(out[i].cpu().numpy(), O.physical_model(h, probs[i % 2])[0]) <= FWD_TOL
        l_ref, g_ref, _ = O.gradient(h, y[i], probs[i % 2])
        assert rel(g[i].cpu().numpy(), g_ref) <= GRAD_TOL
        assert abs(float(loss[i]) / l_ref - 1) <= 1e-4


@pytest.mark.parametrize("n", [1, 8, 9])
def test_joint_update_groups_of_instances(n):
    from paper_2503_20146_amd import PWF
    dev = device()
    geo = dataclasses.replace(S.config_geometry(0), ny=128, nx=128)
    rng = np.random.default_rng(n)
    t = S.diffuser(rng, 128, 128)
    prob = O.make_problem(t, geo)
    psi = [S.phase_object(rng, 128, 128, 4.0, 2.0) for _ in range(n)]
    y = [S.poisson_intensity(O.physical_model(p, prob)[0], (5, i)) for i, p in enumerate(psi)]
    t0 = (t * (1 + 0.05 * rng.standard_normal(t.shape))).astype(np.complex64)
    say(f"joint diffuser step of {n} instances")
    td = to_dev(t0, dev)
    p = gpu_problem(geo, t, dev)
    p.diffuser = td
    out, _ = PWF([p] * n).solve_joint([to_dev(x, dev) for x in y], 6, eta_t=0.5)
    ref, t_ref, _ = O.pwf_joint(y, O.make_problem(t0, geo), 6, 0.5)
    assert rel(td.cpu().numpy(), t_ref) <= 1e-5
    assert np.sqrt(np.mean(np.abs(out[n - 1].cpu().numpy() - ref[n - 1]) ** 2)) <= PHASE_TOL
