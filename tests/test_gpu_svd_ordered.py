"""The ordered form of the Jacobi SVD (block pairs at every n, the QR with a row per
lane, ascending products), which unit cells with wide cuts use, on both sides of
every size at which its launches change: one workgroup with one and two block pairs
(16 | 17, 32 | 33, 48 | 49, 64 rows), cooperative above.  Matrices and bounds are
those of test_gpu_svd_edges.py, which hold for any order."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
from test_gpu_svd_edges import U, dev, matrices  # noqa: E402


def svd(mats, n):
    f = P._lib["_ZN5sictm10launch_svdEiPKPKdPKPdS6_S6_iPvP12ihipStream_tb"]
    f.restype = ctypes.c_int
    w = P._lib["_ZN5sictm19svd_workspace_bytesEii"]
    w.restype = ctypes.c_size_t
    ws = torch.empty(w(len(mats), n), dtype=torch.uint8, device="cuda")
    rd = [dev(m) for m in mats]
    ud, vd = [torch.zeros_like(r) for r in rd], [torch.zeros_like(r) for r in rd]
    sd = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in mats]
    arr = lambda ts: (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])  # noqa: E731
    torch.cuda.synchronize()
    assert f(len(mats), arr(rd), arr(ud), arr(sd), arr(vd), n, ctypes.c_void_p(ws.data_ptr()), None, True) == 0
    torch.cuda.synchronize()
    return [[t.cpu().numpy() for t in x] for x in zip(ud, sd, vd)]


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 96, 97, 105])
def test_ordered(n):
    mats = matrices(n)
    tol = 32 * n ** 1.5 * U + 32 * U
    first = svd(mats, n)
    for m, (u, s, v) in zip(mats, first):
        ref = np.linalg.svd(m, compute_uv=False)
        assert np.all(np.diff(s) <= 0)
        assert np.abs(s - ref).max() <= tol * ref[0]
        assert np.linalg.norm(u.T @ u - np.eye(n), 2) <= tol
        assert np.linalg.norm(v.T @ v - np.eye(n), 2) <= tol
        assert np.linalg.norm((u * s) @ v.T - m, 2) <= tol * ref[0]
    # no sum depends on timing
    again = svd(mats, n)
    assert all(np.array_equal(x, y) for a, b in zip(first, again) for x, y in zip(a, b))
