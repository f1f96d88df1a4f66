"""Products of any width on the split kernel and on both sides of the rule that
sends them there (K = 256, M = 64), through the taped GEMM: forward C = op(A) B
and the cotangents Abar, Bbar, whose products have the other two lengths as K.
Tile edges with a remainder of one, odd widths and leading dimensions, cut and
whole tiles.  Every entry is a sum of L products, so that each side is within
L u of the exact value times the sum of the absolute products (u = 2^-53), and
their difference within twice that; one more u each for the scaling."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402

U = 2.0 ** -53
L = P._lib
_vp = ctypes.c_void_p
L.ctm_tape_check_gemm.restype = ctypes.c_int
L.ctm_tape_check_gemm.argtypes = [ctypes.POINTER(ctypes.c_int), ctypes.POINTER(ctypes.c_long),
                                  ctypes.c_double, _vp, ctypes.c_long, _vp, ctypes.c_long, _vp,
                                  ctypes.c_long, _vp, _vp, _vp]

SHAPES = [(64, 1, 256), (63, 33, 256), (64, 33, 255), (65, 17, 257), (128, 32, 256), (129, 33, 4097),
          (257, 113, 1001), (256, 161, 512), (193, 161, 2049), (1024, 1024, 256), (1025, 1023, 259),
          (2050, 97, 640), (300, 2051, 300), (4097, 257, 256)]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_wide_products(shape, trans):
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A = rng.standard_normal((K, M + 1) if trans else (M, K + 1))   # one column more than is read
    B = rng.standard_normal((K, N + 1))
    Cb = rng.standard_normal((M, N))
    a, b, alpha = (A[:, :M].T if trans else A[:, :K]), B[:, :N], 0.75
    dA, dB, dCb = dev(A), dev(B), dev(Cb)
    gC, gA, gB = torch.zeros_like(dCb), torch.zeros_like(dA), torch.zeros_like(dB)
    dims = (ctypes.c_int * 7)(M, N, K, trans, 1 << 30, 1 << 30, 1)
    st = (ctypes.c_long * 9)(A.shape[1], B.shape[1], 0, N, 0, 1, 0, 0, 0)
    torch.cuda.synchronize()
    assert L.ctm_tape_check_gemm(dims, st, alpha, dA.data_ptr(), A.size, dB.data_ptr(), B.size,
                                 gC.data_ptr(), Cb.size, dCb.data_ptr(), gA.data_ptr(), gB.data_ptr()) == 0

    def check(got, x, y):
        bound = 2 * (x.shape[1] + 1) * U * alpha * (np.abs(x) @ np.abs(y))
        assert np.all(np.abs(got - alpha * (x @ y)) <= bound)

    gA, gB = gA.cpu().numpy(), gB.cpu().numpy()
    check(gC.cpu().numpy(), a, b)
    check(gA[:, :M].T if trans else gA[:, :K], Cb, b.T)
    check(gB[:, :N], a.T, Cb)
    assert not gA[:, M if trans else K].any() and not gB[:, N].any()
