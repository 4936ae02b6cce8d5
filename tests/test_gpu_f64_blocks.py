"""GPU parity of the FP64 pass with the oracle at the edges of its kernels: virtual counts
around the 16-wide blocks and 64-wide tiles, auxiliary counts around the 16-deep chunks
(odd ones among them), few and many pairs, pairs i = j, a mask, active holes, and rows too
long for 32-bit offsets.

FP64 on both sides, sums in another order: 1e-12 of the largest value, a few thousand ulps
for sums of at most ~10^6 terms of random sign (rounding grows with the square root).
"""
import numpy as np
import pytest

import synth
from oracle import dsrg_pt2 as o
from gpu_common import gpu_pass

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _compare(inp, s=0.5, mask=None):
    r = o.pt2_pass_inputs(inp, s, pair_mask=mask) if mask is not None else o.pt2_pass_inputs(inp, s)
    g = gpu_pass(inp, s, pair_mask=mask)
    nc = inp.n_core
    assert abs(g["E"] - (r.energy[0] + r.energy[1])) <= TOL * abs(r.energy[0])
    assert np.abs(g["D"] - r.D_vv).max() <= TOL * np.abs(r.D_vv).max()
    assert np.array_equal(g["D"], g["D"].T)
    # norms are stored in FP32
    assert np.abs(g["pair_tnorm"] - r.pair_tnorm).max() <= 1e-6 * r.pair_tnorm.max()
    e = g["pair_energy"][:nc, :nc]
    assert abs(e.sum() - r.pair_energy[:nc, :nc].sum()) <= TOL * np.abs(r.pair_energy[:nc, :nc]).sum()


@pytest.mark.parametrize("n_vir", [1, 15, 16, 17, 33, 48, 63, 64, 65, 81, 129])
def test_virtual_edges(n_vir):
    print(f"f64 blocks n_vir={n_vir}", flush=True)
    _compare(synth.generate(3, 0, n_vir, 37, seed=n_vir))


@pytest.mark.parametrize("n_aux", [1, 2, 15, 16, 17, 31, 32, 33, 47, 50])
def test_auxiliary_edges(n_aux):
    print(f"f64 blocks n_aux={n_aux}", flush=True)
    _compare(synth.generate(2, 0, 70, n_aux, seed=n_aux))


@pytest.mark.parametrize("n_core,n_act,n_vir", [(1, 0, 30), (1, 2, 66), (9, 4, 49), (70, 0, 5)])
def test_holes(n_core, n_act, n_vir):
    print(f"f64 blocks n_core={n_core} n_act={n_act} n_vir={n_vir}", flush=True)
    _compare(synth.generate(n_core, n_act, n_vir, 41, seed=n_core))


def test_mask():
    inp = synth.generate(8, 0, 67, 35, seed=4)
    m = np.random.default_rng(1).random((8, 8)) < 0.6
    m = (m | m.T).astype(np.uint8)
    print("f64 blocks mask", flush=True)
    _compare(inp, mask=m)


def test_rows_beyond_32_bit_offsets():
    """A 64-row panel of 4.2 million auxiliary functions spans more than 2 GB."""
    print("f64 blocks wide rows", flush=True)
    rng = np.random.default_rng(2)
    n_aux = 4_194_305
    inp = synth.generate(2, 0, 3, 8, seed=5)
    inp = inp.replace(B=0.01 * rng.standard_normal((2, 3, n_aux)))
    _compare(inp)
