"""GPU parity with the oracles of the density terms with active particles, singles and cumulant
where their kernels change form: active spaces of 1, 7, 8, 9 and 12 orbitals (a few particles
or pairs at a time in LDS, more than 64 active pairs), 23 to 26 holes (groups of 24), virtual
counts around the 32-wide tiles of the symmetric amplitudes.

FP64 on both sides, sums of at most ~10^5 terms in another order: 1e-12 of the largest value.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_common import need_gpu
from oracle import a9_active
from oracle import a9_cumulant as cu

pytestmark = pytest.mark.gpu


def _inputs(n_core, n_act, n_vir, n_aux):
    """Inputs and cumulant; an odd active space is an even one without its last orbital."""
    even = n_act + n_act % 2
    inp = synth.generate(n_core, even, n_vir, n_aux, seed=3, active_particles=True)
    lam = synth.active_cumulant(even, 5)
    if n_act < even:
        inp = inp.replace(eps_act=inp.eps_act[:-1], gamma_act=inp.gamma_act[:-1, :-1].copy(), B=inp.B[:-1].copy(),
                          B_act=inp.B_act[:-1, :-1].copy())
        lam = lam[:-1, :-1, :-1, :-1].copy()
    return inp, lam


@pytest.mark.parametrize("sizes", [(0, 1, 1, 3), (2, 1, 31, 17), (16, 7, 5, 20), (15, 8, 33, 33), (17, 9, 11, 19),
                                   (2, 12, 9, 25), (24, 2, 32, 16), (1, 3, 65, 40)], ids=str)
def test_active_terms(sizes):
    print(f"active terms sizes={sizes}", flush=True)
    dp = need_gpu()
    inp, lam = _inputs(*sizes)
    d = dp.upload_inputs(inp)
    opts = dp.make_opts(inp.n_core, inp.n_act, inp.n_vir, inp.n_aux, 0.5)
    zero = lambda: torch.zeros((inp.n_vir, inp.n_vir), dtype=torch.float64, device="cuda")
    D = dp.add_active_particle_density(opts, d["eps_hole"], d["eps_vir"], d["gamma_act"], d["B"], d["B_act"], zero())
    ref = a9_active.active_particle_density(inp.eps_core, inp.eps_act, inp.eps_vir, inp.gamma_act, inp.B, inp.B_act,
                                            0.5)
    assert np.abs(D.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    D = zero()
    lam_d = torch.from_numpy(np.ascontiguousarray(lam)).cuda()
    dp.add_cumulant_singles_density(opts, d["eps_hole"], d["eps_vir"], d["gamma_act"], lam_d, d["B"], d["B_act"], D)
    ref = cu.cumulant_singles_density(inp.eps_core, inp.eps_act, inp.eps_vir, inp.gamma_act, lam, inp.B, inp.B_act, 0.5)
    assert np.abs(D.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
