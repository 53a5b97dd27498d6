"""Forward calls on small grids in batches that do not fill the chip run on plans of their own (four
elements per lane): both sides and their mix against the FP64 oracle, the largest batch that takes
these plans and the smallest that does not.  The solves, the stopping rule and the joint diffuser
step of such batches, which stay on the built-in plans, are held to the same bars."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, rel, say, to_dev

pytestmark = pytest.mark.gpu

FWD_TOL, GRAD_TOL, PHASE_TOL = 1e-5, 1e-4, 1e-3   # the bars of the parity tests


def scene(ny, nx, seed):
    geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx)
    rng = np.random.default_rng(seed)
    psi = S.phase_object(rng, ny, nx, 4.0, 2.0)
    t = S.diffuser(rng, ny, nx)
    prob = O.make_problem(t, geo)
    f, _, _ = O.physical_model(psi, prob)
    return geo, psi, t, prob, S.poisson_intensity(f, (7, seed))


@pytest.mark.parametrize("ny,nx", [(128, 128), (256, 256), (128, 256), (256, 128)])
def test_latency_plans_match_oracle(ny, nx):
    from paper_2503_20146_amd import PWF
    dev = device()
    geo, psi, t, prob, y = scene(ny, nx, ny + nx)
    batch = PWF([gpu_problem(geo, t, dev)])
    half = (0.5 * psi).astype(np.complex64)
    say(f"latency plans {ny} x {nx}")
    f_ref, _, _ = O.physical_model(half.astype(np.complex128), prob)
    assert rel(batch.forward([to_dev(half, dev)])[0].cpu().numpy(), f_ref) <= FWD_TOL
    loss, g, _ = batch.gradient([to_dev(half, dev)], [to_dev(y, dev)])
    l_ref, g_ref, _ = O.gradient(half.astype(np.complex128), y, prob)
    assert rel(g[0].cpu().numpy(), g_ref) <= GRAD_TOL
    assert abs(float(loss[0]) / l_ref - 1) <= 2e-5 * np.linalg.norm(f_ref) / np.linalg.norm(y - f_ref)
    out, _ = batch.solve([to_dev(y, dev)], 30)
    psi_ref, _, _ = O.pwf(y, prob, 30)
    assert np.sqrt(np.mean(np.abs(out[0].cpu().numpy() - psi_ref) ** 2)) <= PHASE_TOL


def test_stopping_rule_and_joint_step_on_latency_plans():
    from paper_2503_20146_amd import PWF
    dev = device()
    geo, psi, t, prob, y = scene(128, 256, 5)
    say("latency plans: stopping rule and joint diffuser step")
    tol = 1.0 - 1e-4
    out, _, done = PWF([gpu_problem(geo, t, dev)]).solve([to_dev(y, dev)], 60, corr_tol=tol, return_iters=True)
    psi_ref, hist, _ = O.pwf(y, prob, 60, corr_tol=tol)
    assert done[0] == len(hist) < 60
    assert np.sqrt(np.mean(np.abs(out[0].cpu().numpy() - psi_ref) ** 2)) <= PHASE_TOL
    t0 = (t * (1 + 0.05 * np.random.default_rng(3).standard_normal(t.shape))).astype(np.complex64)
    td = to_dev(t0, dev)
    p = gpu_problem(geo, t, dev)
    p.diffuser = td
    psi_j, _ = PWF([p]).solve_joint([to_dev(y, dev)], 8, eta_t=0.5)
    ref, t_ref, _ = O.pwf_joint([y], O.make_problem(t0, geo), 8, 0.5)
    assert np.sqrt(np.mean(np.abs(psi_j[0].cpu().numpy() - ref[0]) ** 2)) <= PHASE_TOL
    assert rel(td.cpu().numpy(), t_ref) <= 1e-5


@pytest.mark.parametrize("count", [64, 65])
def test_batches_around_the_limit(count):
    """64 fields of 128^2 take the latency plans, 65 the others: both match one instance on its
    own to FP32 rounding (phase tolerance), and every instance of the batch is the same."""
    from paper_2503_20146_amd import PWF
    import torch
    dev = device()
    geo, psi, t, prob, y = scene(128, 128, 9)
    p, yd = gpu_problem(geo, t, dev), to_dev(y, dev)
    say(f"batch of {count} x 128^2")
    out, hist = PWF([p] * count).solve([yd] * count, 10)
    one, hist1 = PWF([p]).solve([yd], 10)
    assert all(torch.equal(out[0], o) for o in out)
    assert float((out[0] - one[0]).abs().square().mean().sqrt()) <= 1e-5
    assert torch.allclose(hist[count - 1], hist1[0], rtol=1e-5)


@pytest.mark.parametrize("count", [64, 65])
def test_forward_around_the_limit(count):
    """64 fields of 128^2 take the latency plans, 65 the others."""
    from paper_2503_20146_amd import PWF
    import torch
    dev = device()
    geo, psi, t, prob, _ = scene(128, 128, 11)
    p = gpu_problem(geo, t, dev)
    f_ref, _, _ = O.physical_model(psi, prob)
    say(f"forward of {count} x 128^2")
    f = PWF([p] * count).forward([to_dev(psi.astype(np.complex64), dev)] * count)
    assert all(torch.equal(f[0], g) for g in f)
    assert rel(f[0].cpu().numpy(), f_ref) <= FWD_TOL
