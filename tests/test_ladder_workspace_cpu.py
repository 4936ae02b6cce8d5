"""The ladder's workspace does not hold another copy of the amplitudes: it stays within the blocks of
integrals (16 GB, or 1024 n^2 doubles and 2 GB), 2 GB of split amplitudes and the transformed inputs."""
import os

import pytest

import paper_2312_07008_amd as dp
from paper_2312_07008_amd import _lib, api


@pytest.mark.parametrize("n,n_aux,n_amp,n_kept", [(1000, 2500, 7500, 0), (1000, 2500, 11000, 0), (400, 1600, 400, 0),
                                                  (60, 200, 65535, 0), (2048, 4000, 16, 0), (500, 1500, 20000, 300)])
def test_workspace_bound(n, n_aux, n_amp, n_kept):
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("library not built")
    dp.load()
    m = n_kept or n
    blocks = max(16.0e9, 1024 * 8.0 * m * m + 2.0e9)
    inputs = 8.0 * (n * m * n_aux + m * m * n_aux + n_amp * n * m + n_amp * m * m) if n_kept else 2.0e9
    assert api.pp_ladder_workspace_size(n, n_aux, n_amp, n_kept) <= blocks + inputs + 8.0 * m * m + 4096
