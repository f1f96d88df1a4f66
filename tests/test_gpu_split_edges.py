"""The split product (stream-K) at the edges of its tiles: every width class
of N, row counts on both sides of the 128-, 192- and 256-row tiles, K with a
full and a partial last slice, ranges shorter than a tile, and leading
dimensions of either parity.  A length-K dot product in any order is within
(K + 2) u of the sum of |terms|; twice that covers the reference's own
rounding."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402

U = 2.0 ** -53
CASES = [(M, N, K) for N, M, K in [
    (1, 127, 241), (2, 128, 256), (15, 129, 257), (16, 255, 272), (17, 256, 300), (33, 257, 255),
    (48, 191, 511), (49, 385, 512), (72, 1024, 264), (80, 130, 1023), (87, 515, 515), (96, 64, 400),
    (105, 500, 500), (112, 1, 999), (113, 193, 250), (128, 192, 321), (129, 384, 256), (159, 385, 270),
    (160, 577, 1000)]]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("M,N,K", CASES)
def test_split_edges(M, N, K):
    rng = np.random.default_rng(M + 1000 * N)
    trans = [0, 1, 1]
    lda = max(M, K) + (max(M, K) & 1)                 # the entry point asks for an even one
    A = [rng.standard_normal((K if t else M, lda)) for t in trans]
    B = [rng.standard_normal((K, N)) for _ in trans]
    scratch = torch.empty(P.gemm_f64_split_scratch_bytes() // 8, dtype=torch.float64, device="cuda")
    Ad, Bd = [dev(a) for a in A], [dev(b) for b in B]
    for ncu in (256, 5):
        Cd = [torch.full((M, N), 7.0, dtype=torch.float64, device="cuda") for _ in trans]
        assert P.gemm_f64_split(Ad, Bd, Cd, M, N, K, trans, scratch, ncu=ncu, lda=lda)
        torch.cuda.synchronize()
        for a, t, b, c in zip(A, trans, B, Cd):
            op = a[:, :M].T if t else a[:, :K]
            bound = 2 * (K + 2) * U * (np.abs(op) @ np.abs(b))
            assert np.all(np.abs(c.cpu().numpy() - op @ b) <= bound)


@pytest.mark.parametrize("M,N,K,trans", [(301, 87, 301, 0), (301, 87, 301, 1), (515, 33, 259, 0),
                                         (193, 121, 247, 1), (1875, 87, 1875, 0)])
def test_split_with_odd_rows(M, N, K, trans):
    """Odd leading dimensions on both sides, through the tape's GEMM."""
    L = P._lib
    L.ctm_tape_check_gemm.restype = ctypes.c_int
    vp = ctypes.c_void_p
    L.ctm_tape_check_gemm.argtypes = [ctypes.POINTER(ctypes.c_int), ctypes.POINTER(ctypes.c_long),
                                      ctypes.c_double, vp, ctypes.c_long, vp, ctypes.c_long, vp,
                                      ctypes.c_long, vp, vp, vp]
    rng = np.random.default_rng(M)
    lda = M if trans else K
    assert lda % 2 == 1 and N % 2 == 1
    A = rng.standard_normal((K, M) if trans else (M, K))
    B, bar = rng.standard_normal((K, N)), rng.standard_normal((M, N))
    Ad, Bd, bard = dev(A), dev(B), dev(bar)
    C, Ab, Bb = torch.zeros(M, N, dtype=torch.float64, device="cuda"), torch.zeros_like(Ad), torch.zeros_like(Bd)
    dims = (ctypes.c_int * 7)(M, N, K, trans, 1 << 30, 1 << 30, 1)
    strides = (ctypes.c_long * 9)(lda, N, 0, N, 0, 1, 0, 0, 0)
    st = L.ctm_tape_check_gemm(dims, strides, 1.0, Ad.data_ptr(), A.size, Bd.data_ptr(), B.size,
                               C.data_ptr(), C.numel(), bard.data_ptr(), Ab.data_ptr(), Bb.data_ptr())
    assert st == 0
    op = A.T if trans else A
    for got, x, y in [(C, op, B), (Bb, op.T, bar),
                      (Ab, B if trans else bar, (bar if trans else B).T)]:
        bound = 2 * (x.shape[1] + 2) * U * (np.abs(x) @ np.abs(y))
        assert np.all(np.abs(got.cpu().numpy() - x @ y) <= bound)
