"""Shell correlation over half spectra (pwf_fsc.hip) against the FP64 oracle at the sizes where
its passes change: the smallest side (one element per lane, 16 row pairs per workgroup), 256
(per-pass twiddle tables, two chunks per row), 1024 in 2-D (64-lane rows), rows that are their
own mirror (ky, kz = 0 and n/2), both parts, and inputs at the ends of the FP32 range."""

import numpy as np
import pytest

import oracle as O
from gpu_helpers import device, say, to_dev

pytestmark = pytest.mark.gpu

# |FSC_GPU - FSC_oracle| per shell: spectra carry a relative FP32 rounding of a few 1e-7 each
TOL = 1e-5


def fields(n, dims, seed):
    rng = np.random.default_rng(seed)
    shape = (n,) * dims
    s = rng.standard_normal(shape, dtype=np.float32)
    return [((s + 0.7 * rng.standard_normal(shape, dtype=np.float32))
             + 1j * (2.0 * s + rng.standard_normal(shape, dtype=np.float32))).astype(np.complex64) for _ in range(2)]


@pytest.mark.parametrize("n,dims,part", [(128, 2, 1), (128, 3, 1), (256, 3, 0), (256, 2, 1), (1024, 2, 0)])
def test_shells_match_oracle(n, dims, part):
    from paper_2503_20146_amd import shell_correlation
    dev = device()
    a, b = fields(n, dims, 10 * n + dims)
    pick = (lambda g: g.imag) if part else (lambda g: g.real)
    say(f"shells {n}^{dims} part {part}")
    got = np.array(shell_correlation(to_dev(a, dev), to_dev(b, dev), part=part))
    assert np.max(np.abs(got - O.shell_correlation(pick(a), pick(b)))) <= TOL


@pytest.mark.parametrize("sa,sb", [(2.0 ** -120, 1.0), (2.0 ** 115, 2.0 ** -110), (1.0, 2.0 ** 120)])
def test_shells_at_the_ends_of_the_fp32_range(sa, sb):
    """Powers of two are exact, so the correlation is that of the unscaled inputs."""
    from paper_2503_20146_amd import shell_correlation
    dev = device()
    a, b = fields(128, 2, 5)
    say(f"shells, inputs times {sa:g}, {sb:g}")
    got = np.array(shell_correlation(to_dev((np.float32(sa) * a).astype(np.complex64), dev),
                                     to_dev((np.float32(sb) * b).astype(np.complex64), dev), part=0))
    assert np.max(np.abs(got - O.shell_correlation(a.real, b.real))) <= TOL


def test_empty_and_nonfinite_inputs_give_nan():
    from paper_2503_20146_amd import shell_correlation
    dev = device()
    a, b = fields(128, 2, 6)
    say("shells of a zero field and of a field with a NaN")
    assert np.all(np.isnan(shell_correlation(to_dev(0 * a, dev), to_dev(b, dev), part=0)))
    a[3, 5] = np.nan
    assert np.all(np.isnan(shell_correlation(to_dev(a, dev), to_dev(b, dev), part=0)))
