"""Householder QR on the eight-wavefront leaves, on both sides of every size at
which they begin, end or change their register height (192 | 193 and 384 | 385
rows of one leaf, 256 | 257 rows of a leaf, 8 | 9 four-wavefront leaves, 8 | 9
eight-wavefront ones), one panel and several, narrow last panels.  Checked by
what defines the factorisation, within the same small multiple of sqrt(N) k u of
the norms involved, u = 2^-53.  Rows that do not split into leaves of k to 192
rows are refused, also where the taller leaves would hold them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402

SHAPES = [(192, 32), (193, 1), (193, 32), (193, 160), (255, 33), (256, 31), (257, 64), (257, 192), (383, 65),
          (384, 5), (384, 32), (385, 32), (1151, 20), (1152, 33), (1281, 40), (2049, 97), (2500, 105),
          (3072, 64), (3073, 17)]


@pytest.mark.parametrize("N,k", SHAPES)
def test_qr_wide_edges(N, k):
    W = [S.gaussian_block(N, k, 90 + i) for i in range(3)]
    W[1] = W[1] * np.logspace(0, -12, k)                     # graded columns
    W[2][:, k // 2] = 0.0                                    # a zero column
    if k > 3:
        W[2][:, k - 1] = W[2][:, 0] - 3.0 * W[2][:, 1]       # a dependent one
    Wd = [torch.from_numpy(np.ascontiguousarray(w)).cuda() for w in W]
    if not any(N // nb >= k and -(-N // nb) <= 192 for nb in range(1, N // k + 1)):
        with pytest.raises(P.CtmError):
            P.qr_f64(Wd)
        return
    P.qr_f64(Wd)
    torch.cuda.synchronize()
    u = 2.0 ** -53
    tol = 8 * np.sqrt(N) * k * u + 16 * u
    for w, d in zip(W, Wd):
        q = d.cpu().numpy()
        nrm = np.linalg.norm(w)
        r = q.T @ w
        assert np.all(np.isfinite(q))
        assert np.linalg.norm(q.T @ q - np.eye(k)) <= tol
        assert np.linalg.norm(np.tril(r, -1)) <= tol * nrm
        assert np.all(np.diag(r) >= -tol * nrm)
        assert np.linalg.norm(q @ r - w) <= tol * nrm
