"""GPU ladder where its blocks of pairs (a, b), b <= a, change form: matrices around the 32-wide
tiles of the symmetric split, few and many amplitude matrices, contractions split over
workgroups, and a space so large that the pairs of one a are formed in parts and contracted in
several blocks.

Against R^p = sum_Q B^Q T^p B^Q^T in FP64 on the CPU; sums of n^2 n_aux terms of random sign in
another order, 1e-12 of the largest element (rounding 2^-53 sqrt(terms) ~ 1e-13).
"""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


def _check(n, n_aux, n_amp, n_kept=0):
    dp = need_gpu()
    g = torch.Generator().manual_seed(n)
    B = torch.randn(n, n, n_aux, generator=g, dtype=torch.float64)
    B = B + B.transpose(0, 1)
    T = torch.randn(n_amp, n, n, generator=g, dtype=torch.float64)
    X = torch.linalg.qr(torch.randn(n, n, generator=g, dtype=torch.float64))[0].contiguous() if n_kept else None
    R = dp.pp_ladder(B.cuda(), T.cuda(), X.cuda(), n_kept) if n_kept else dp.pp_ladder(B.cuda(), T.cuda())
    if n_kept:
        Xk = X[:, :n_kept]
        B = torch.einsum("ax,abq,by->xyq", Xk, B, Xk)
        T = Xk.T @ T @ Xk
    ref = sum(B[:, :, q] @ T @ B[:, :, q].T for q in range(n_aux))
    assert (R.cpu() - ref).abs().max() <= 1e-12 * ref.abs().max()


@pytest.mark.parametrize("n", [1, 2, 16, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("n_amp", [1, 65])
def test_small_spaces(n, n_amp):
    print(f"ladder blocks n={n} n_amp={n_amp}", flush=True)
    _check(n, 7, n_amp)


@pytest.mark.parametrize("n,n_aux,n_amp,n_kept", [(90, 40, 300, 71), (200, 17, 3, 0), (40, 33, 500, 33)])
def test_split_contractions(n, n_aux, n_amp, n_kept):
    print(f"ladder blocks n={n} n_aux={n_aux} n_amp={n_amp} n_kept={n_kept}", flush=True)
    _check(n, n_aux, n_amp, n_kept)


def test_pairs_of_one_row_in_parts():
    print("ladder blocks n=650", flush=True)
    _check(650, 2, 2)
