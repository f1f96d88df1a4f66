"""The workspaces that ctm_qr_f64 and ctm_svd_f64 keep between calls: sizes that
grow, shrink and exceed what is kept (also when no block fits any more), several
threads on streams of their own, and a context destroyed in between.  Every result
has the bits of a first call on the same input; what a device keeps is bounded."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402

QR = [(1, 64, 16), (3, 500, 40), (8, 2500, 105), (1, 1024, 72), (8, 20000, 160), (2, 300, 97)]
SVD = [5, 64, 97, 130]


def qr(count, N, k, stream=None):
    W = [torch.from_numpy(S.gaussian_block(N, k, 40 + i)).cuda() for i in range(count)]
    torch.cuda.synchronize()
    P.qr_f64(W, stream)
    return [w.cpu().numpy() for w in W]


def svd(n, stream=None):
    A = [torch.from_numpy(S.gaussian_block(n, n, 50 + i)).cuda() for i in range(4)]
    U, V = [torch.zeros_like(a) for a in A], [torch.zeros_like(a) for a in A]
    s = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in A]
    torch.cuda.synchronize()
    P.svd_f64(A, U, s, V, stream)
    return [x.cpu().numpy() for x in U + s + V]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def test_sizes_in_turn_and_bound():
    ref = {c: qr(*c) for c in QR}
    for c in QR + QR[::-1]:
        assert same(qr(*c), ref[c])
    # destroying a context gives the blocks back; they are at most 256 MiB
    ctx = P.Ctm(P.Config(d=2, D=2, chi=4, p=2, n_si=1),
                torch.from_numpy(S.product_plus_noise_site(2, 2, 3)).cuda())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx.close()
    assert torch.cuda.mem_get_info()[0] - before <= (256 << 20) + (64 << 20)
    assert same(qr(*QR[2]), ref[QR[2]])


def test_threads_and_streams():
    qref, sref = {c: qr(*c) for c in QR[:4]}, {n: svd(n) for n in SVD}
    bad = []

    def work(i):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for r in range(6):
                c, n = QR[(i + r) % 4], SVD[(i + r) % 4]
                if not same(qr(*c, st), qref[c]) or not same(svd(n, st), sref[n]):
                    bad.append((i, r, c, n))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
