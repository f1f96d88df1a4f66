"""The adjoint of a move at block widths on both sides of the register rows of the
triangular inverse (64 | 65 and 128 | 129 columns), which are also remainders of its
16 columns per workgroup and of the batched transposes' 32, against the reverse-mode
reference.  Both sides lose the condition of the QR's R (below 1e5 for these blocks)
and the smallest relative gap of the singular values (above 1e-4) from u = 1e-16: 1e-7;
the bound is ten times that, and a wrong column would be off by its own size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle.adjoint as J  # noqa: E402
import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402


def rel(a, b):
    return np.abs(np.asarray(a) - np.asarray(b)).max() / np.abs(np.asarray(b)).max()


@pytest.mark.parametrize("chi,p", [(29, 4), (60, 4), (60, 5), (121, 7), (121, 8)])
def test_move_vjp_edges(chi, p):
    D, n_si = 2, 1
    Dl, N, k = D * D, chi * D * D, chi + p
    A = S.product_plus_noise_site(2, D, 11, noise=1.0)
    C = [S.gaussian_block(chi, chi, 60 + i) for i in range(4)]
    T = [S.gaussian_block(chi * Dl, chi, 70 + i).reshape(chi, Dl, chi) for i in range(4)]
    X = [np.linalg.qr(S.gaussian_block(N, k, 20 + b))[0] for b in range(4)]
    Y = [np.linalg.qr(S.gaussian_block(N, k, 30 + b))[0] for b in range(4)]
    ctx = P.Ctm(P.Config(d=2, D=D, chi=chi, p=p, n_si=n_si), torch.from_numpy(A).cuda())
    state = ctx.pack_state(C, T, np.stack(X), np.stack(Y))
    rng = np.random.default_rng(5)
    bars = ([rng.standard_normal((chi, chi)) for _ in range(4)],
            [rng.standard_normal((chi, Dl, chi)) for _ in range(4)],
            [rng.standard_normal(x.shape) for x in X], [rng.standard_normal(y.shape) for y in Y])
    bar = ctx.pack_state(bars[0], bars[1], np.stack(bars[2]), np.stack(bars[3]))
    in_bar, _, site_bar = ctx.move_vjp(torch.from_numpy(state), torch.from_numpy(bar))
    ib = in_bar.cpu().numpy()
    ib[-4] = chi                      # counters of a cotangent are zero; unpack at chi
    g = ctx.unpack_state(ib)
    gC, gT, gX, gY, gA = J.move_vjp(C, T, X, Y, A, bars, chi, n_si)
    for got, ref in ((g["C"], gC), (g["T"], gT), (g["X"], gX), (g["Yt"], gY)):
        assert max(rel(a, b) for a, b in zip(got, ref)) <= 1e-6
    assert rel(site_bar.cpu().numpy(), gA) <= 1e-6
