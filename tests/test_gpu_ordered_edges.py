"""The ordered products and QR that unit cells with wide cuts use, at the edges of
their rules: cut ranges on both sides of 16 slices and of N = 128 and 160, unaligned
operands and rows (which are not cut), whole tiles on both sides of the size that
takes them, inner batches, remainders of K, accumulation and an output map.  Every
sum over K products of either side is within K u of the exact value times the sum of
the absolute products, u = 2^-53, so their difference within twice that.  An element
of a product that is not cut has the bits of the same element computed in a product
of few columns (ascending k whatever the tile).  The QR is checked by what defines
it, as in test_gpu_qr_edges.py."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402

U = 2.0 ** -53
VP, I, LG = ctypes.c_void_p, ctypes.c_int, ctypes.c_long


class Batch(ctypes.Structure):
    _fields_ = [("A", VP * 8), ("B", VP * 8), ("C", VP * 8), ("trans", I * 8), ("count", I), ("M", I), ("N", I), ("K", I),
                ("lda", LG), ("ldb", LG), ("cdiv_m", I), ("cs_m1", LG), ("cs_m0", LG), ("cdiv_n", I), ("cs_n1", LG),
                ("cs_n0", LG), ("nbatch", I), ("a_bs", LG), ("b_bs", LG), ("c_bs", LG), ("alpha", ctypes.c_double),
                ("accumulate", I), ("split", I)]


def product(A, B, C, M, N, K, trans, lda, ldb, scratch, accumulate=0, nbatch=1, bs=(0, 0, 0), m_map=None, ldc=None):
    f = P._lib["_ZN5sictm19launch_gemm_orderedERKNS_9GemmBatchEPdiP12ihipStream_t"]
    f.restype = I
    g = Batch()
    g.count, g.M, g.N, g.K, g.lda, g.ldb, g.nbatch, g.alpha, g.accumulate = len(A), M, N, K, lda, ldb, nbatch, 0.75, accumulate
    g.cdiv_m, g.cs_m1, g.cs_m0 = m_map or (1 << 30, 0, ldc or N)
    g.cdiv_n, g.cs_n1, g.cs_n0 = 1 << 30, 0, 1
    g.a_bs, g.b_bs, g.c_bs = bs
    for i in range(len(A)):
        g.A[i], g.B[i], g.C[i], g.trans[i] = A[i].data_ptr(), B[i].data_ptr(), C[i].data_ptr(), trans
    torch.cuda.synchronize()
    assert f(ctypes.byref(g), VP(scratch.data_ptr() if scratch is not None else None), 256, None) == 0
    torch.cuda.synchronize()


def scratch():
    return torch.empty(P.gemm_f64_split_scratch_bytes(), dtype=torch.uint8, device="cuda")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


SHAPES = [
    # M, N, K, problems: cut from 16 slices on, N <= 160
    (97, 97, 241, 1), (97, 97, 240, 1), (193, 128, 256, 2), (193, 129, 257, 2), (383, 160, 999, 3), (384, 161, 999, 3),
    (2500, 105, 2500, 4), (105, 105, 2500, 4), (1, 2, 300, 1),
    # whole tiles from 128 of them on, and the tile kernels
    (2500, 2500, 100, 1), (2440, 1153, 17, 1), (2440, 1153, 16, 1), (8200, 625, 31, 2), (100, 2500, 100, 8), (300, 64, 50, 2),
]


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_products(shape, trans):
    M, N, K, n = shape
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    for pad in (0, 1):   # an odd leading dimension of A is not cut, an odd one of B is
        ra, ca = ((K, M) if trans else (M, K))
        A = [rng.standard_normal((ra, ca + (ca + pad) % 2)) for _ in range(n)]
        B = [rng.standard_normal((K, N + pad)) for _ in range(n)]
        C0 = rng.standard_normal((M, N))
        for acc in (0, 1):
            C = [dev(C0) for _ in range(n)]
            product([dev(a) for a in A], [dev(b) for b in B], C, M, N, K, trans, A[0].shape[1], N + pad, scratch(), acc)
            for a, b, c in zip(A, B, C):
                a = a[:, :M].T if trans else a[:, :K]
                b = b[:, :N]
                want = 0.75 * (a @ b) + acc * C0
                bound = 2 * (K + 2) * U * (np.abs(a) @ np.abs(b) + acc * np.abs(C0))
                assert np.all(np.abs(c.cpu().numpy() - want) <= bound)


@pytest.mark.parametrize("M,N,K", [(2500, 1300, 100), (1300, 2500, 33), (12000, 625, 50)])
def test_whole_tiles_have_the_bits_of_the_tile_kernels(M, N, K):
    rng = np.random.default_rng(5)
    A, B = dev(rng.standard_normal((M, K))), dev(rng.standard_normal((K, N)))
    C, D = (torch.zeros(M, N, dtype=torch.float64, device="cuda") for _ in range(2))
    product([A], [B], [C], M, N, K, 0, K, N, None)
    for n0 in range(0, N, 64):   # at most 64 columns: tile kernels
        w = min(64, N - n0)
        product([A], [B[:, n0:]], [D[:, n0:]], M, w, K, 0, K, N, None, ldc=N)
    assert torch.equal(C, D)


def test_unaligned_operands_are_not_cut():
    """Operands 8 bytes off: whole sums, the bits of the same product without scratch."""
    M, N, K = 500, 110, 600
    rng = np.random.default_rng(6)
    a, b = dev(rng.standard_normal(M * K + 1)), dev(rng.standard_normal(K * N + 1))
    C, D, E = (torch.zeros(M, N, dtype=torch.float64, device="cuda") for _ in range(3))
    product([a[1:]], [b[1:]], [C], M, N, K, 0, K, N, scratch())
    product([a[1:]], [b[1:]], [D], M, N, K, 0, K, N, None)
    assert torch.equal(C, D)
    x, y = a[1:].cpu().numpy().reshape(M, K), b[1:].cpu().numpy().reshape(K, N)
    assert np.all(np.abs(C.cpu().numpy() - 0.75 * (x @ y)) <= 2 * (K + 2) * U * (np.abs(x) @ np.abs(y)))
    # cut where they are aligned: the same values to the bound
    p, q = a[1:].clone(), b[1:].clone()
    product([p], [q], [E], M, N, K, 0, K, N, scratch())
    assert np.all(np.abs(E.cpu().numpy() - 0.75 * (x @ y)) <= 2 * (K + 2) * U * (np.abs(x) @ np.abs(y)))


@pytest.mark.parametrize("M,N,K,nb", [(500, 300, 90, 25), (40, 30, 20, 7)])
def test_inner_batches_and_output_map(M, N, K, nb):
    rng = np.random.default_rng(7)
    A, B = rng.standard_normal((nb, M, K)), rng.standard_normal((nb, K, N))
    C = torch.zeros(nb, M, N, dtype=torch.float64, device="cuda")
    # rows (i, j), j < 10, stored j-major
    product([dev(A)], [dev(B)], [C], M, N, K, 0, K, N, scratch(), nbatch=nb, bs=(M * K, K * N, M * N),
            m_map=(10, N, M // 10 * N))
    got = C.cpu().numpy().reshape(nb, 10, M // 10, N).transpose(0, 2, 1, 3).reshape(nb, M, N)
    for a, b, c in zip(A, B, got):
        assert np.all(np.abs(c - 0.75 * (a @ b)) <= 2 * (K + 2) * U * (np.abs(a) @ np.abs(b)))


@pytest.mark.parametrize("N,k", [(97, 97), (192, 33), (200, 97), (385, 100), (855, 101), (1500, 192), (2500, 105), (8300, 33)])
def test_ordered_qr(N, k):
    f = P._lib["_ZN5sictm17launch_qr_orderedEiPKPdiiPvP12ihipStream_t"]
    w = P._lib["_ZN5sictm26qr_ordered_workspace_bytesEiii"]
    f.restype, w.restype = I, ctypes.c_size_t
    W = [S.gaussian_block(N, k, 60 + i) for i in range(3)]
    W[1] = W[1] * np.logspace(0, -10, k)
    W[2][:, k // 2] = 0.0
    D = [dev(x) for x in W]
    ws = torch.empty(w(3, N, k), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    r = f(3, (VP * 3)(*[d.data_ptr() for d in D]), N, k, VP(ws.data_ptr()), None)
    torch.cuda.synchronize()
    ok = P._lib["_ZN5sictm10qr_plan_okEii"]
    ok.restype = ctypes.c_bool
    assert (r == 0) == ok(N, k)
    if r:
        return
    tol = 8 * np.sqrt(N) * k * U + 16 * U
    for x, d in zip(W, D):
        q = d.cpu().numpy()
        assert np.linalg.norm(q.T @ q - np.eye(k)) <= tol
        t, nrm = q.T @ x, np.linalg.norm(x)
        assert np.linalg.norm(np.tril(t, -1)) <= tol * nrm
        assert np.all(np.diag(t) >= -tol * nrm)
        assert np.linalg.norm(q @ t - x) <= tol * nrm
