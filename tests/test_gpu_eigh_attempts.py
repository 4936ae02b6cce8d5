"""The eigensolver where its one-launch reduction does not come through: a workgroup of it that
never runs (the others give up and a second attempt takes one launch per column), and a launch that
is refused.  Against LAPACK at the bars of test_gpu_eigh_paths.py, and with one buffer for the matrix
and the vectors, which the attempt that is given up has to leave alone.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

AUTO, MISSED, REFUSED = 0, 1, 2


def _run(A, path, in_place):
    dp = need_gpu()
    from paper_2312_07008_amd import api
    n = A.shape[0]
    a = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    w = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    Z = a if in_place else torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    ws = torch.full((api.fno_truncate_workspace_size(n),), 255, dtype=torch.uint8, device="cuda")
    attempts = ctypes.c_int(0)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    st = dp.load().dfpt2_eigh_sym_path(ptr(a), ctypes.c_int64(n), ptr(w), ptr(Z), ptr(ws), ctypes.c_size_t(ws.numel()),
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), path,
                                       ctypes.byref(attempts))
    torch.cuda.synchronize()
    assert st == 0
    return w.cpu().numpy(), Z.cpu().numpy(), attempts.value


# one workgroup, few and many of them, the widest rows
@pytest.mark.parametrize("n,path", [(65, AUTO), (129, MISSED), (300, MISSED), (1200, MISSED), (2048, MISSED),
                                    (4, REFUSED), (129, REFUSED), (300, REFUSED), (1200, AUTO)])
@pytest.mark.parametrize("in_place", [False, True])
def test_attempts(n, path, in_place):
    print(f"eigh n={n} path={path} in_place={in_place}", flush=True)
    X = np.random.default_rng(n).standard_normal((n, n))
    A = X + X.T
    w, Z, attempts = _run(A, path, in_place)
    assert attempts == (2 if path == MISSED else 1)
    wref = np.linalg.eigvalsh(A)
    nrm, grow = np.abs(wref).max(), max(1.0, np.sqrt(n) / 4)
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - wref).max() <= 1e-13 * nrm * grow
    assert np.abs(A @ Z - Z * w[None, :]).max() <= 1e-12 * nrm * grow
    assert np.abs(Z.T @ Z - np.eye(n)).max() <= 1e-11
