"""GPU parity with the oracle where the kernels at a pass's ends change form: tile-partial
counts and batches around the rule that reduces them in the last kernel, with and without a
mask, and the screen's features at row and column counts around their 16-row and 64-column
workgroups.

Energies and densities: FP64 on both sides, sums in another order, 1e-12 of the largest value.
Features are stored in FP32 (half an ulp is 6e-8 of the value) from FP64 logarithms of sums of
at most a few hundred positive terms (1e-13).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import dsrg_pt2 as o
from oracle import screening as sc
from gpu_common import gpu_pass, need_gpu

pytestmark = pytest.mark.gpu


# 192 virtuals are 6 tile partials a pair, 193 are 10 (a launch of their own)
@pytest.mark.parametrize("n_vir", [4, 64, 192, 193])
@pytest.mark.parametrize("batch", [0, 8, 15])
@pytest.mark.parametrize("masked", [False, True])
def test_pass_ends(n_vir, batch, masked):
    print(f"pass ends n_vir={n_vir} batch={batch} masked={masked}", flush=True)
    inp = synth.generate(5, 2, n_vir, 33, seed=n_vir)
    mask = None
    if masked:
        m = np.random.default_rng(7).random((7, 7)) < 0.7
        m = m | m.T
        m[5:, :] = m[:, 5:] = True
        m[0, 1] = m[1, 0] = False
        mask = m
    r = o.pt2_pass_inputs(inp, 0.5, pair_mask=mask)
    g = gpu_pass(inp, 0.5, pair_mask=mask, pair_batch=batch)
    assert abs(g["E"] - (r.energy[0] + r.energy[1])) <= 1e-12 * abs(r.energy[0])
    assert np.abs(g["D"] - r.D_vv).max() <= 1e-12 * np.abs(r.D_vv).max()
    assert np.abs(g["pair_tnorm"] - r.pair_tnorm).max() <= 1e-6 * r.pair_tnorm.max()
    core = g["pair_energy"][:5, :5]
    assert np.abs(core - r.pair_energy[:5, :5]).max() <= 1e-12 * np.abs(r.pair_energy[:5, :5]).max()
    assert np.isnan(g["pair_energy"][5:, :]).all() and np.isnan(g["pair_energy"][:, 5:]).all()
    if masked:
        assert core[0, 1] == 0.0 and g["pair_tnorm"][0, 1] == 0.0


@pytest.mark.parametrize("n_core,n_vir,n_aux", [(1, 1, 1), (2, 15, 63), (3, 16, 64), (5, 17, 65), (4, 33, 200)])
def test_features(n_core, n_vir, n_aux):
    print(f"features n_core={n_core} n_vir={n_vir} n_aux={n_aux}", flush=True)
    dp = need_gpu()
    inp = synth.generate(n_core, 0, n_vir, n_aux, seed=n_aux)
    ref = sc.pair_quantities(inp, 0.5)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    opts = dp.make_opts(n_core, 0, n_vir, n_aux, 0.5)
    f, ls = dp.pairscreen_features(opts, dev(inp.eps_hole), dev(inp.eps_vir), dev(inp.B))
    np.testing.assert_allclose(f.cpu().numpy(), ref["feats"], rtol=1.2e-7, atol=1e-12)
    np.testing.assert_allclose(ls.cpu().numpy()[:, 0], ref["log_gw"], rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(ls.cpu().numpy()[:, 1], ref["log_gu"], rtol=1e-12, atol=1e-12)
