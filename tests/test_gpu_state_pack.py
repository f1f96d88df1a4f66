"""The state vector on the device equals the one on the host bit for bit: while the
environment grows (zeros behind its tensors), before any blocks exist, with pending
start blocks, with current ones, and where more segments than one launch takes are
packed (a unit cell's state there and back)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402


@pytest.mark.parametrize("D,chi,p,blocks", [(2, 5, 3, False), (2, 5, 3, True), (3, 17, 4, True)])
def test_state_device_equals_host(D, chi, p, blocks):
    ctx = P.Ctm(P.Config(d=2, D=D, chi=chi, p=p, n_si=1),
                torch.from_numpy(S.product_plus_noise_site(2, D, 7)).cuda())
    if blocks:
        N, k = chi * D * D, min(chi + p, chi * D * D)
        X, Y = (torch.stack([torch.from_numpy(S.gaussian_block(N, k, o + b)) for b in range(4)]).cuda()
                for o in (20, 30))
        ctx.set_isometries(X, Y)
    for _ in range(5):
        dev = ctx.get_state_device().cpu().numpy()
        assert np.array_equal(dev, ctx.get_state())
        ctx.move()


@pytest.mark.parametrize("shape", [(1, 1), (2, 2), (3, 3)])
def test_cell_state_round_trip(shape):
    Lx, Ly = shape
    D, chi, p = 2, 6, 2
    cell = P.Cell(P.CellConfig(Lx=Lx, Ly=Ly, d=2, D=D, chi=chi, p=p, n_si=1),
                  torch.stack([torch.from_numpy(S.product_plus_noise_site(2, D, 3 + i))
                               for i in range(Lx * Ly)]).cuda())
    state = torch.from_numpy(np.random.default_rng(4).standard_normal(cell.state_size())).cuda()
    cell.set_state_device(state)
    assert torch.equal(cell.get_state_device(), state)
