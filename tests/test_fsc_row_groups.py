"""What the shell-sum kernel (fsc_shell_kernel in pwf_fsc.hip) reads and how it weighs it, modelled in
FP64 on the CPU: half spectra of two rows at a time with kx = 0 and n/2 packed at position 0, the
rows (+-ky, +-kz) taken together (a row that is its own mirror twice at half weight), kx > 0 counted
for -kx, position 0 separated with the mirrored row.  The sums must be those of a bincount over the
whole spectra, for random fields, to FP64 rounding."""

import itertools

import numpy as np
import pytest


def half_spectra(a, n, dims):
    """fsc_rows_kernel and fsc_cols_kernel: twice the row transforms of two rows at once, then y (and z)."""
    rows = a.reshape(-1, n)
    c = np.fft.fft(rows[0::2] + 1j * rows[1::2], axis=1)
    k = np.arange(n // 2)
    cm = np.conj(c[:, (n - k) % n])
    x = np.empty((rows.shape[0], n // 2), complex)
    x[0::2] = c[:, k] + cm
    x[1::2] = (c[:, k] - cm) / 1j
    x[0::2, 0] = 2 * (c[:, 0].real + 1j * c[:, n // 2].real)
    x[1::2, 0] = 2 * (c[:, 0].imag + 1j * c[:, n // 2].imag)
    x = x.reshape(a.shape[:-1] + (n // 2,))
    return np.fft.fftn(x, axes=tuple(range(dims - 1)))


def model_sums(A, B, n, dims):
    h, nsh = n // 2, n // 2 + 1
    A, B = (x.reshape((n,) * (dims - 1) + (h,)) if dims == 3 else x[None] for x in (A, B))
    out = np.zeros((3, nsh))

    def add(kappa, a, b, w):
        if kappa < nsh:
            out[:, kappa] += w * np.array([a.real * b.real + a.imag * b.imag, abs(a) ** 2, abs(b) ** 2])

    for kz, ky, kx in itertools.product(range(h + 1) if dims == 3 else (0,), range(h + 1), range(h)):
        rows = [((n - kz) % n if i & 2 else kz, (n - ky) % n if i & 1 else ky) for i in range(4 if dims == 3 else 2)]
        wr = (0.5 if ky % h == 0 else 1.0) * (0.5 if dims == 3 and kz % h == 0 else 1.0)
        r2 = ky * ky + kz * kz
        kappa = int(np.rint(np.sqrt(kx * kx + r2)))
        if kx:
            for r in rows:
                add(kappa, A[r][kx], B[r][kx], 2.0 * wr)
            continue
        for i in range(len(rows) // 2):
            u, m = rows[i], rows[len(rows) - 1 - i]
            x0 = [X[u][0] + np.conj(X[m][0]) for X in (A, B)]
            xn = [(X[u][0] - np.conj(X[m][0])) / 1j for X in (A, B)]
            add(kappa, *x0, 0.5 * wr)
            add(int(np.rint(np.sqrt(h * h + r2))), *xn, 0.5 * wr)
    return out


@pytest.mark.parametrize("n,dims", [(8, 2), (32, 2), (8, 3), (16, 3)])
def test_row_groups_and_packed_column(n, dims):
    rng = np.random.default_rng(n + dims)
    a, b = rng.standard_normal((2,) + (n,) * dims)
    b += 0.5 * a
    f = np.fft.fftfreq(n, 1 / n)
    r = np.rint(np.sqrt(sum(g * g for g in np.meshgrid(*[f] * dims, indexing="ij")))).astype(int)
    Fa, Fb = np.fft.fftn(a), np.fft.fftn(b)
    want = [np.bincount(r.ravel(), v.ravel(), minlength=n)[:n // 2 + 1]
            for v in (np.real(np.conj(Fa) * Fb), np.abs(Fa) ** 2, np.abs(Fb) ** 2)]
    got = model_sums(half_spectra(a, n, dims), half_spectra(b, n, dims), n, dims) / 4   # (every spectrum is doubled)
    assert np.allclose(got, want, rtol=1e-12, atol=1e-12 * want[1].max())
