"""Small float64 products, whose workgroups split K over their wavefronts, on
both sides of every remainder (16 rows, 16 columns, 16 and 128 of K) and of the
rule's line, both orientations, odd leading dimensions, alpha and accumulation,
non-finite values in rows and columns next to the ones read.  Each entry is a sum
of K products, so that either side is within K u of the exact value times the sum
of the absolute products (u = 2^-53); two more u for alpha and the accumulation."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402

U = 2.0 ** -53
SHAPES = [(1, 1, 1), (1, 17, 2), (15, 16, 15), (16, 15, 16), (17, 33, 17), (31, 20, 32), (32, 49, 33),
          (33, 64, 127), (48, 81, 128), (20, 5, 129), (64, 79, 257), (243, 32, 243), (105, 105, 2500),
          (512, 37, 515), (7, 1000, 64), (1000, 7, 64), (1025, 41, 97), (1024, 80, 1024)]


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_products(shape, trans):
    M, N, K = shape
    count, alpha = 3, -1.25
    rng = np.random.default_rng(M + 5 * N + 11 * K)
    A = [np.full((K, M + 1) if trans else (M, K + 1), np.nan) for _ in range(count)]
    B = [np.full((K, N + 1), np.inf) for _ in range(count)]
    for a, b in zip(A, B):
        a[:, :-1] = rng.standard_normal((a.shape[0], a.shape[1] - 1))
        b[:, :-1] = rng.standard_normal((K, N))
    C = [rng.standard_normal((M, N)) for _ in range(count)]
    dA, dB, dC = ([torch.from_numpy(x).cuda() for x in y] for y in (A, B, C))
    for accumulate in (0, 1):
        before = [c.cpu().numpy() for c in dC]
        P.gemm_f64(dA, dB, dC, M, N, K, trans_a=trans, lda=A[0].shape[1], ldb=N + 1, alpha=alpha,
                   accumulate=accumulate)
        torch.cuda.synchronize()
        for a, b, c0, c in zip(A, B, before, dC):
            x, y = (a[:, :-1].T if trans else a[:, :-1]), b[:, :-1]
            ref = alpha * (x @ y) + (c0 if accumulate else 0.0)
            mass = abs(alpha) * (np.abs(x) @ np.abs(y))
            bound = 2 * (K + 2) * U * (mass + (np.abs(c0) if accumulate else 0.0))
            assert np.all(np.abs(c.cpu().numpy() - ref) <= bound)
