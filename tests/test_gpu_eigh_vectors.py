"""Accuracy of the GPU eigensolver's vectors where a stage is formed differently for speed than
plain inverse iteration and a reflector at a time.

Twisted factorizations, on the tridiagonal matrix (-1, 2, -1), whose eigenpairs are known in
closed form and which the reduction leaves as it is.  A solve is exact for matrix entries off by
independent roundings: about five of rms 0.29 eps per position, of entries up to ||T|| / 2, meet two
vectors with entries of rms n^(-1/2) and give 0.65 eps ||T|| / sqrt(n) along a neighbour at the
distance `gap`, summed over the neighbours on both sides 1.5 times that; four sigma for the largest
of n vectors is 4 eps ||T|| / (sqrt(n) gap).  Twice that is allowed, for the orthonormalization at the
end, and 8 eps for the last operations.  A common error of the shift, such as an
eigenvalue's own rounding, would count with the full eps ||T|| / gap.

Back-transformation, on random symmetric matrices, whose vectors have entries of n^(-1/2) and
residuals that the eigenvalues' rounding hardly shows in.  One rounding of rms eps / sqrt(12) per
entry and block of 16 reflectors, and as much again in the products, add up to 0.29 * 2 * eps / 4 over
n / 16 blocks (n^(1/2) / 4 times n^(-1/2)); A - w magnifies it by at most 1.2 ||A||, and the largest of
n^2 entries lies at six sigma: 1.04 eps ||A||, with a margin 1.1.  A rounding per reflector, or per term of
a sum over the rows, adds up to several times that.
"""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


def _eigh(A):
    dp = need_gpu()
    w, Z = dp.eigh_sym(torch.from_numpy(np.ascontiguousarray(A)).cuda())
    return w.cpu().numpy(), Z.cpu().numpy()


# four vectors a wave up to 2044 rows, one a wave beyond
@pytest.mark.parametrize("n", [600, 1200, 2049])
def test_vectors_of_isolated_eigenvalues(n):
    print(f"eigenvectors of the second difference n={n}", flush=True)
    _, Z = _eigh(2 * np.eye(n) - np.eye(n, k=1) - np.eye(n, k=-1))
    L = np.longdouble
    k = np.arange(1, n + 1, dtype=L)
    pi = 4 * np.arctan(L(1))
    S = np.sqrt(L(2) / (n + 1)) * np.sin(pi * k[:, None] * k[None, :] / (n + 1))
    step = np.diff(2 - 2 * np.cos(pi * k / (n + 1))).astype(float)
    gap = np.minimum(np.r_[np.inf, step], np.r_[step, np.inf])
    err = np.sqrt(((Z * np.sign((S * Z).sum(0)) - S) ** 2).sum(0)).astype(float)
    assert np.all(err <= 8 * EPS * 4 / (np.sqrt(n) * gap) + 8 * EPS)


@pytest.mark.parametrize("n", [600, 1200])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_residuals_of_random_matrices(n, seed):
    print(f"residuals of a random matrix n={n} seed={seed}", flush=True)
    X = np.random.default_rng(seed).standard_normal((n, n))
    A = X + X.T
    w, Z = _eigh(A)
    assert np.abs(A @ Z - Z * w[None, :]).max() <= 1.1 * EPS * np.abs(w).max()
