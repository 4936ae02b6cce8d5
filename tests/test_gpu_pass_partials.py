"""GPU parity with the oracle on either side of the number of tile partials (pairs times partials a
pair, 4096) up to which the last kernel of a pass reduces them itself, with and without a mask
that moves a pass across it.  FP64 on both sides, sums in another order: 1e-12 of the largest value.
"""
import numpy as np
import pytest

import synth
from oracle import dsrg_pt2 as o
from gpu_common import gpu_pass

pytestmark = pytest.mark.gpu


# 60 virtuals are one partial a pair, 70 three, 130 six: 4095 and 4186, 3978 and 4134, 3996 and 4218
@pytest.mark.parametrize("n_core,n_vir", [(90, 60), (91, 60), (51, 70), (52, 70), (36, 130), (37, 130)])
@pytest.mark.parametrize("masked", [False, True])
def test_partials(n_core, n_vir, masked):
    print(f"tile partials n_core={n_core} n_vir={n_vir} masked={masked}", flush=True)
    inp = synth.generate(n_core, 0, n_vir, 17, seed=n_core)
    mask = None
    if masked:
        m = np.random.default_rng(1).random((n_core, n_core)) < 0.9
        mask = m | m.T
    r = o.pt2_pass_inputs(inp, 0.5, pair_mask=mask)
    g = gpu_pass(inp, 0.5, pair_mask=mask, pair_batch=65535)
    assert abs(g["E"] - (r.energy[0] + r.energy[1])) <= 1e-12 * abs(r.energy[0])
    assert np.abs(g["D"] - r.D_vv).max() <= 1e-12 * np.abs(r.D_vv).max()
    assert np.abs(g["pair_energy"] - r.pair_energy).max() <= 1e-12 * np.abs(r.pair_energy).max()
    assert np.abs(g["pair_tnorm"] - r.pair_tnorm).max() <= 1e-6 * r.pair_tnorm.max()
