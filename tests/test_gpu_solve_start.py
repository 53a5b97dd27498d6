"""The first iterations of a solve, which take their zero state from no memory: 0 to 3 iterations in a
workspace that an earlier solve of other data has left full, one grid shape and several (per-class and
merged launches), with the stopping rule on, against the FP64 oracle."""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synthetic as S
from gpu_helpers import device, gpu_problem, say, to_dev

pytestmark = pytest.mark.gpu

PHASE_TOL = LOSS_TOL = 1e-3   # the parity tests' bar


@pytest.mark.parametrize("iters", [0, 1, 2, 3])
@pytest.mark.parametrize("shapes,merged,tol", [([(128, 256)], 0, 0.0), ([(128, 128)], 0, 0.9999999),
                                               ([(512, 512), (512, 1024)], 0, 0.0),
                                               ([(512, 512), (512, 1024)], 1, 0.0)])
def test_first_iterations(shapes, merged, tol, iters):
    from paper_2503_20146_amd import PWF
    import paper_2503_20146_amd as P
    dev = device()
    rng = np.random.default_rng(17)
    probs, refs, ys, other = [], [], [], []
    for i, (ny, nx) in enumerate(shapes):
        geo = dataclasses.replace(S.config_geometry(0), ny=ny, nx=nx)
        t = S.diffuser(rng, ny, nx)
        refs.append(O.make_problem(t, geo))
        f = O.physical_model(S.phase_object(rng, ny, nx, 4.0, 2.0), refs[-1])[0]
        ys.append(S.poisson_intensity(f, (13, i)))
        other.append(to_dev(np.ascontiguousarray(ys[-1][::-1, ::-1]), dev))
        probs.append(gpu_problem(geo, t, dev))
    say(f"{iters} iterations of {shapes}, merged {merged}, tol {tol}")
    P.set_merged_launch(bool(merged))
    try:
        batch = PWF(probs)
        batch.solve(other, 4)
        out, hist = batch.solve([to_dev(y, dev) for y in ys], iters, corr_tol=tol)
        for i, ref in enumerate(refs):
            want, losses, _ = O.pwf(ys[i], ref, iters)
            assert np.sqrt(np.mean(np.abs(out[i].cpu().numpy() - want) ** 2)) <= PHASE_TOL
            if iters:
                assert np.allclose(hist[i].cpu().numpy(), losses, rtol=LOSS_TOL)
    finally:
        P.set_merged_launch(False)
