"""Jacobi SVD on both sides of every size at which its kernels change (one
workgroup up to n = 96, or 128 for values only, the block-pair kernels above;
register heights of 16 rows; blocks of 13 to 16 columns), with odd sizes,
graded, rank-deficient and scaled matrices.  The bounds are those of a
backward stable SVD: |s - s_ref|, |U^T U - I|, |V^T V - I| and |U S V^T - A|
within a small multiple of n^(3/2) u of the largest singular value (or of
one), u = 2^-53."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402

U = 2.0 ** -53
SIZES = [1, 2, 3, 5, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 87, 95, 96, 97, 105,
         112, 113, 128, 129, 144, 161, 192]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def matrices(n):
    rng = np.random.default_rng(n)
    q = lambda: np.linalg.qr(rng.standard_normal((n, n)))[0]  # noqa: E731
    flat = rng.standard_normal((n, n))
    graded = (q() * np.logspace(0, -14, n)) @ q()
    low = flat[:, : max(1, n // 3)] @ rng.standard_normal((max(1, n // 3), n))
    pairs = (q() * np.repeat(np.linspace(2, 1, (n + 1) // 2), 2)[:n]) @ q()   # equal pairs
    return [flat, graded, low, pairs, 1e-140 * flat, 1e140 * graded]


@pytest.mark.parametrize("n", SIZES)
def test_svd_edges(n):
    mats = matrices(n)
    rd = [dev(m) for m in mats]
    ud, vd = [torch.zeros_like(r) for r in rd], [torch.zeros_like(r) for r in rd]
    sd = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in mats]
    P.svd_f64(rd, ud, sd, vd)
    torch.cuda.synchronize()
    tol = 32 * n ** 1.5 * U + 32 * U
    for m, u, s, v in zip(mats, ud, sd, vd):
        u, s, v = u.cpu().numpy(), s.cpu().numpy(), v.cpu().numpy()
        ref = np.linalg.svd(m, compute_uv=False)
        assert np.all(np.diff(s) <= 0)
        assert np.abs(s - ref).max() <= tol * ref[0]
        assert np.linalg.norm(u.T @ u - np.eye(n), 2) <= tol
        assert np.linalg.norm(v.T @ v - np.eye(n), 2) <= tol
        assert np.linalg.norm((u * s) @ v.T - m, 2) <= tol * ref[0]


@pytest.mark.parametrize("n", SIZES)
def test_svd_values_only_edges(n):
    mats = matrices(n)
    sd = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in mats]
    P.svd_f64([dev(m) for m in mats], None, sd, None)
    torch.cuda.synchronize()
    for m, s in zip(mats, sd):
        ref = np.linalg.svd(m, compute_uv=False)
        assert np.abs(s.cpu().numpy() - ref).max() <= (32 * n ** 1.5 * U + 32 * U) * ref[0]
