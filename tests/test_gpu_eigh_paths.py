"""GPU eigensolver against LAPACK at the sizes where its kernels change: the smallest
matrices, one workgroup (n <= 128), the resident form (n <= 2048) and one launch per column
beyond it, the back-transformation's register blocks, and spectra whose vectors take the
twisted factorizations, the pivoted inverse iteration, or both.

Bars as in test_gpu_fp64.py: eigenvalues 1e-13 ||A|| max(1, sqrt(n) / 4) (rounding of the
reduction, sqrt(n) of its backward error), residuals 1e-12 of the same, orthogonality
1e-11.
"""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


def _check(A):
    dp = need_gpu()
    n = A.shape[0]
    w, Z = dp.eigh_sym(torch.from_numpy(np.ascontiguousarray(A)).cuda())
    w, Z = w.cpu().numpy(), Z.cpu().numpy()
    wref = np.linalg.eigvalsh(A)
    nrm, grow = np.abs(wref).max(), max(1.0, np.sqrt(n) / 4)
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - wref).max() <= 1e-13 * nrm * grow
    assert np.abs(A @ Z - Z * w[None, :]).max() <= 1e-12 * nrm * grow
    assert np.abs(Z.T @ Z - np.eye(n)).max() <= 1e-11


@pytest.mark.parametrize("n", [4, 7, 8, 63, 64, 65, 127, 128, 129, 256, 257, 513, 1281, 2048, 2049])
def test_sizes(n):
    print(f"eigh n={n}", flush=True)
    X = np.random.default_rng(n).standard_normal((n, n))
    _check(X + X.T)


@pytest.mark.parametrize("n", [96, 200])
@pytest.mark.parametrize("gap", [1e-13, 1e-11, 1e-9, 3e-8, 1e-6])
def test_close_eigenvalues(n, gap):
    """Runs of eigenvalues `gap` ||A|| apart beside isolated ones."""
    print(f"eigh close eigenvalues n={n} gap={gap}", flush=True)
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = np.concatenate([1 + gap * np.arange(9), 2 + gap * np.arange(2), 3 + rng.random(n - 11)]) * (1e3 / 4)
    A = (Q * lam) @ Q.T
    _check(0.5 * (A + A.T))


@pytest.mark.parametrize("scale", [1e-120, 1e120])
@pytest.mark.parametrize("n", [50, 300])
def test_scaled_and_split(n, scale):
    """Far from unit norm, with zero off-diagonal blocks and off-diagonals of 1e-40."""
    print(f"eigh scaled n={n} scale={scale}", flush=True)
    X = np.random.default_rng(n).standard_normal((n, n))
    A = X + X.T
    h = n // 2
    A[h:, :h] = A[:h, h:] = 0.0
    A[h, h - 1] = A[h - 1, h] = 1e-40
    _check(A * scale)
