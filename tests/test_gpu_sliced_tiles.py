"""GPU parity with the oracle of the BF16 and INT8 sliced pair products where their 128 x 128
tiles change form: a last tile with at most 64 columns (or rows) deals its blocks to the waves
in another way.  Contractions long enough for the pipelined loop and shorter ones.

The slices leave 2^-34 (BF16) and 2^-33 (INT8, five digits) of a row's largest elements per
product, at most a few 1e-10 of the largest pair energy or density element at these sizes; a
block in the wrong place changes them by order one.  Bound: 1e-8.
"""
import numpy as np
import pytest

import synth
from oracle import dsrg_pt2 as o
from gpu_common import gpu_pass

pytestmark = pytest.mark.gpu

BF16, INT8 = 1, 3


@pytest.mark.parametrize("precision", [BF16, INT8], ids=["bf16", "int8"])
@pytest.mark.parametrize("n_vir", [1, 33, 64, 65, 96, 128, 129, 160, 192, 193, 257])
@pytest.mark.parametrize("n_aux", [33, 300])
def test_last_tile(precision, n_vir, n_aux):
    print(f"sliced tiles precision={precision} n_vir={n_vir} n_aux={n_aux}", flush=True)
    inp = synth.generate(3, 0, n_vir, n_aux, seed=n_vir)
    r = o.pt2_pass_inputs(inp, 0.5)
    g = gpu_pass(inp, 0.5, precision=precision)
    assert np.abs(g["pair_energy"] - r.pair_energy).max() <= 1e-8 * np.abs(r.pair_energy).max()
    assert np.abs(g["pair_tnorm"] - r.pair_tnorm).max() <= 1e-6 * r.pair_tnorm.max()
    assert np.abs(g["D"] - r.D_vv).max() <= 1e-8 * np.abs(r.D_vv).max()
