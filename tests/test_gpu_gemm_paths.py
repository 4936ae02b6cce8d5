"""GPU parity of the FP64 GEMM's tiles, splits and offset ranges, through the entry
points that run on it: the ladder (edges of the 64- and 128-wide tiles, odd leading
dimensions, rows too far apart for 32-bit offsets) and the active-particle density
(contractions split over workgroups).

Both sides are FP64 and differ only in the order of their sums: 1e-12 of the largest
element (a few hundred ulps for sums of at most ~10^6 terms of random sign, whose
rounding grows with the square root of their number).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import a9_active, ladder
from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n_v,n_aux,n_amp", [(63, 16, 1), (64, 15, 65), (65, 33, 3), (128, 17, 2), (129, 31, 4)])
def test_ladder_at_tile_edges(n_v, n_aux, n_amp):
    dp = need_gpu()
    inp = synth.ladder_inputs(n_v, n_aux, n_amp, seed=n_v)
    print(f"ladder tile edges n_v={n_v} n_aux={n_aux} n_amp={n_amp}", flush=True)
    ref = ladder.pp_ladder(inp.B_vv, inp.T)
    R = dp.pp_ladder(_dev(inp.B_vv), _dev(inp.T)).cpu().numpy()
    assert np.abs(R - ref).max() <= TOL * np.abs(ref).max()


def test_ladder_rows_beyond_32_bit_offsets():
    """Sixteen rows of X^T B (n_kept n_aux doubles apart) span more than 2 GB."""
    dp = need_gpu()
    n_v, n_aux, n_amp, n_kept = 42, 421_001, 2, 40
    g = torch.Generator(device="cuda").manual_seed(3)
    z = torch.randn(n_v, n_v, n_aux, generator=g, device="cuda", dtype=torch.float64)
    B = (z + z.transpose(0, 1)).contiguous()
    del z
    T = torch.randn(n_amp, n_v, n_v, generator=g, device="cuda", dtype=torch.float64)
    q, _ = np.linalg.qr(np.random.default_rng(5).standard_normal((n_v, n_v)))
    X = _dev(q[:, :n_kept])
    print(f"ladder wide rows n_v={n_v} n_aux={n_aux}", flush=True)
    R = dp.pp_ladder(B, T, X, n_kept)
    S = (B.view(n_v * n_v, n_aux) @ B.view(n_v * n_v, n_aux).T).view(n_v, n_v, n_v, n_v)  # (ac|bd), plain FP64
    S = S.permute(0, 2, 1, 3).reshape(n_v * n_v, n_v * n_v)
    P = X @ X.T
    Tp = P @ T @ P
    ref = X.T @ (S @ Tp.reshape(n_amp, -1).T).T.reshape(n_amp, n_v, n_v) @ X
    assert float((R - ref).abs().max()) <= TOL * float(ref.abs().max())


@pytest.mark.parametrize("n_core,n_act,n_v", [(20, 6, 33), (21, 4, 64), (18, 6, 130)])
def test_split_contraction(n_core, n_act, n_v):
    dp = need_gpu()
    inp = synth.generate(n_core, n_act, n_v, 37, seed=n_v, active_particles=True)
    print(f"split contraction n_core={n_core} n_act={n_act} n_v={n_v}", flush=True)
    ref = a9_active.active_particle_density(inp.eps_core, inp.eps_act, inp.eps_vir, inp.gamma_act, inp.B, inp.B_act, 0.5)
    d = dp.upload_inputs(inp)
    D = torch.zeros(n_v, n_v, dtype=torch.float64, device="cuda")
    opts = dp.make_opts(n_core, n_act, n_v, 37, 0.5)
    dp.add_active_particle_density(opts, d["eps_hole"], d["eps_vir"], d["gamma_act"], d["B"], d["B_act"], D)
    ref = 0.5 * (ref + ref.T)
    assert np.abs(D.cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()
