"""Householder QR at the edges of its layout: one leaf and many, leaves on
both sides of 64 and 128 rows (the register heights of the panel kernel),
nodes of 2 to 8 children in one to three tree levels, panels narrower than
32 columns, zero and dependent columns, and magnitudes near the ends of the
exponent range.  Checked by what defines the factorisation (orthonormal Q,
R = Q^T W upper triangular with R_ii >= 0, W = Q R); Householder QR satisfies
each within a small multiple of sqrt(N) k u of the norms involved, u = 2^-53.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402

SHAPES = [
    # N, k: leaves x rows, panels
    (1, 1), (7, 7), (32, 20), (64, 16), (65, 17),            # one leaf of 1 .. 65 rows
    (128, 31), (129, 32), (192, 33), (192, 192), (191, 130),  # one leaf, several panels
    (256, 100), (300, 97), (384, 192),                       # 2 leaves (2 children)
    (400, 32), (520, 64), (700, 65),                         # 3 to 5 leaves
    (1024, 16), (1153, 48), (1300, 160),                     # 8 and 9 leaves: a second level
    (8300, 33), (12500, 5),                                  # 64 and 97 leaves: three levels
]


def check(w, q):
    N, k = w.shape
    u = 2.0 ** -53
    tol = 8 * np.sqrt(N) * k * u + 16 * u
    assert np.all(np.isfinite(q))
    assert np.linalg.norm(q.T @ q - np.eye(k)) <= tol
    r = q.T @ w
    nrm = np.linalg.norm(w)
    assert np.linalg.norm(np.tril(r, -1)) <= tol * nrm
    assert np.all(np.diag(r) >= -tol * nrm)
    assert np.linalg.norm(q @ r - w) <= tol * nrm


@pytest.mark.parametrize("N,k", SHAPES)
def test_qr_edges(N, k):
    W = [S.gaussian_block(N, k, 70 + i) for i in range(3)]
    W[1] = W[1] * np.logspace(0, -12, k)                     # graded columns
    W[2][:, k // 2] = 0.0                                    # a zero column
    if k > 3:
        W[2][:, k - 1] = W[2][:, 0] - 3.0 * W[2][:, 1]       # a dependent one
    Wd = [torch.from_numpy(np.ascontiguousarray(w)).cuda() for w in W]
    P.qr_f64(Wd)
    torch.cuda.synchronize()
    for w, q in zip(W, Wd):
        check(w, q.cpu().numpy())


@pytest.mark.parametrize("scale", [1e-145, 1e145])
def test_qr_extreme_magnitudes(scale):
    w = S.gaussian_block(500, 40, 9)
    d = torch.from_numpy(w * scale).cuda()
    P.qr_f64([d])
    torch.cuda.synchronize()
    check(w, d.cpu().numpy())
