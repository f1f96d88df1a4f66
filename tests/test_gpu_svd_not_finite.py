"""SVDs of matrices that hold NaN or infinity beside finite ones: every rank by
counting stays a permutation, so the kernels read and write only their own memory,
the finite matrices keep the bits they have without the others, and the singular
values of the others show that they were not finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402


def svd(mats):
    n = mats[0].shape[0]
    A = [torch.from_numpy(np.ascontiguousarray(m)).cuda() for m in mats]
    U, V = [torch.zeros_like(a) for a in A], [torch.zeros_like(a) for a in A]
    s = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in A]
    P.svd_f64(A, U, s, V)
    return [[x.cpu().numpy() for x in t] for t in zip(U, s, V)]


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("n", [1, 5, 48, 96, 97, 130, 192])
def test_beside_finite(n, value):
    good = [S.gaussian_block(n, n, 7), S.gaussian_block(n, n, 8)]
    one, many = S.gaussian_block(n, n, 9), S.gaussian_block(n, n, 10)
    one[n // 2, n // 3] = value
    many[:, ::2] = value
    want = svd(good)
    got = svd([good[0], one, good[1], many])
    for i, j in ((0, 0), (2, 1)):
        assert all(np.array_equal(x, y) for x, y in zip(got[i], want[j]))
    for i in (1, 3):
        assert not np.all(np.isfinite(got[i][1]))
