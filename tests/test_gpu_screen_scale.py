"""The training step's divisions by the number of samples, on a network of zeros and one target, where
every other operation is exact in FP32: loss = sum e^2 / n and the gradient of the last bias
sum 2 e / n, at numbers of samples whose reciprocal times the number is not 1 in FP32.  Exact.
"""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

F = np.float32


@pytest.mark.parametrize("n", [82, 94, 188, 3004, 3010])
def test_divisions(n):
    assert F(n) * (F(1) / F(n)) != F(1) and F(n / 2) * (F(2) / F(n)) != F(1)
    print(f"training step scale n={n}", flush=True)
    dp = need_gpu()
    W, m, v = (torch.zeros(dp.pairscreen_num_params(), device="cuda") for _ in range(3))
    f = torch.zeros(n, 5, device="cuda")
    losses = dp.pairscreen_train(W, m, v, f, torch.full((n,), -1.0, device="cuda"), 1, 1e-3)
    assert float(losses[0]) == 1.0  # n squares of 1, over n
    W.zero_(), m.zero_(), v.zero_()
    dp.pairscreen_train(W, m, v, f, torch.full((n,), -n / 2.0, device="cuda"), 1, 1e-3)
    assert float(m[-1]) == float((F(1) - F(0.9)) * F(n))  # n terms 2 (n / 2) / n = 1
    assert not bool(m[:-1].any())
