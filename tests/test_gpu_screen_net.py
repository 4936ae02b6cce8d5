"""GPU parity of the pair-screen network's kernels with the FP64 oracle at the sizes where
their tiles end: fewer samples than a tile, its edges, and more tiles than workgroups.

FP32 against FP64.  A prediction sums 64 products of magnitude ~1 with two tanh of a few
ulps in front: 64 x 6e-8 x 4 = 2e-5.  A gradient sums d pred times factors of at most ~4;
with sum |d pred| = 1 its terms add up to at most ~4 in magnitude, and at most ~256 of them
meet in one chain: 4 x 256 x 6e-8 = 6e-5.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import screening as sc
from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


def _inputs(n):
    rng = np.random.default_rng(n)
    X = np.stack([rng.uniform(-1.5, -0.3, n), rng.uniform(-1.5, -0.3, n), 2.6 + 0.1 * rng.standard_normal(n),
                  -0.02 * rng.random(n), 0.1 * rng.standard_normal(n)], 1).astype(np.float32)
    W = synth.mlp_init(3).astype(np.float32)
    return X, W, rng


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 1000, 33000])
def test_forward_and_backward(n):
    dp = need_gpu()
    X, W, rng = _inputs(n)
    dout = rng.standard_normal(n).astype(np.float32)
    dout /= np.abs(dout).sum()
    print(f"network forward and backward n={n}", flush=True)
    f, w = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    pred, cache = dp.pairscreen_mlp_forward(w, f, want_cache=True)
    plain, _ = dp.pairscreen_mlp_forward(w, f)
    dW = dp.pairscreen_mlp_backward(w, f, cache, torch.from_numpy(dout).cuda())
    ref, c = sc.mlp_forward(W.astype(np.float64), X.astype(np.float64))
    g = sc.mlp_backward(W.astype(np.float64), c, dout.astype(np.float64))
    assert torch.equal(pred, plain)
    assert np.abs(pred.cpu().numpy() - ref).max() <= 2e-5
    assert np.abs(cache.cpu().numpy() - np.concatenate([c["h1"], c["h2"]], 1)).max() <= 2e-5
    assert np.abs(dW.cpu().numpy() - g).max() <= 6e-5


@pytest.mark.parametrize("n", [1, 65, 2000, 33000])
def test_training_step_is_forward_backward_adam(n):
    """One training step against the same step from the separate entry points."""
    dp = need_gpu()
    X, W, rng = _inputs(n)
    y = rng.standard_normal(n).astype(np.float32)
    print(f"network training step n={n}", flush=True)
    f, t = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    a, b = torch.from_numpy(W).cuda(), torch.from_numpy(W).cuda()
    ma, va, mb, vb = (torch.zeros_like(a) for _ in range(4))
    loss = dp.pairscreen_train(a, ma, va, f, t, 1, 3e-3)
    pred, cache = dp.pairscreen_mlp_forward(b, f, want_cache=True)
    dW = dp.pairscreen_mlp_backward(b, f, cache, 2.0 * (pred - t) / n)
    dp.pairscreen_adam_step(b, dW, mb, vb, 1, 3e-3)
    r = (pred - t).double()
    assert abs(float(loss[0]) - float((r * r).mean())) <= 1e-5 * float((r * r).mean())
    # sum |d pred| <= 2 max |r|: the bound above, on the first moment 0.1 dW
    assert float((ma - mb).abs().max()) <= 0.1 * 6e-5 * 2 * float(r.abs().max())
    assert float((a - b).abs().max()) <= 2 * 3e-3  # Adam's first step is lr sign(dW)
    same = dW.abs() > 6e-5 * 2 * float(r.abs().max())
    assert float((a - b)[same].abs().max()) <= 1e-6 if bool(same.any()) else True
