"""GPU ladder in the full space with more amplitude matrices than are split at a time (2 GB of them),
in one block of pairs and in several, against R^p = sum_Q B^Q T^p B^Q^T in FP64 for amplitudes on both
sides of every cut: sums of n^2 n_aux terms of random sign in another order, 1e-12 of the largest element.
"""
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


# 61035, 10014 and 6250 matrices are split at a time; 200 virtuals are two blocks of pairs
@pytest.mark.parametrize("n,n_amp", [(64, 65535), (64, 61036), (64, 61035), (158, 20003), (200, 6251)])
def test_amplitudes_in_parts(n, n_amp):
    print(f"ladder chunks n={n} n_amp={n_amp}", flush=True)
    dp = need_gpu()
    g = torch.Generator(device="cuda").manual_seed(n)
    B = torch.randn(n, n, 5, generator=g, dtype=torch.float64, device="cuda")
    B = B + B.transpose(0, 1)
    T = torch.randn(n_amp, n, n, generator=g, dtype=torch.float64, device="cuda")
    R = dp.pp_ladder(B, T)
    cut = int(2.0e9 // (8 * n * n))
    at = sorted({p for c in range(0, n_amp + cut, cut) for p in (c - 1, c, c + 1) if 0 <= p < n_amp} | {n_amp - 1})
    Bc, Tc = B.cpu(), T[at].cpu()
    ref = sum(Bc[:, :, q] @ Tc @ Bc[:, :, q].T for q in range(5))
    assert (R[at].cpu() - ref).abs().max() <= 1e-12 * ref.abs().max()
