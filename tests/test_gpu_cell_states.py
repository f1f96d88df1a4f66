"""One SI iteration of a unit cell with wide cuts (k > 96) from a given state.

Such an iteration amplifies the last bits of its sums to elements that differ by
up to 3e-7 of the rms, so its state is defined by the order of those sums: it is
compared with recorded elements of the state that the same order gives
(``golden/cell_states.npz``, written by ``golden/make_cell_states.py``).  The path
has no sum whose order depends on timing, so the elements are the same numbers.
"""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "cell_states.npz")
# Lx, Ly, D, chi, p, seed: the benchmark's sites and size, and narrower legs with
# odd k and N, one site per column and per row
CASES = [(2, 2, 5, 100, 5, 1), (2, 2, 5, 100, 5, 2), (2, 2, 3, 95, 6, 3), (1, 2, 4, 93, 8, 4), (2, 1, 2, 120, 9, 5)]
SAMPLES = 1024


def prepare(Lx, Ly, D, chi, p, seed):
    """A cell and a random state of it."""
    r = np.random.default_rng(seed)
    ns, d, Dl = Lx * Ly, 2, D * D
    N, k = chi * Dl, chi + p
    A = {2: 0.35, 3: 0.2, 4: 0.15, 5: 0.1}[D] * (2.0 * r.random((ns, d, D, D, D, D)) - 1.0)
    A[:, 0, 0, 0, 0, 0] += 1.0
    parts = []
    for _ in range(ns):
        for shape in [(chi, chi)] * 4 + [(chi, Dl, chi)] * 4:
            t = r.standard_normal(shape)
            parts.append(t.ravel() / np.linalg.norm(t))
    parts.append(r.standard_normal(8 * ns * N * k))
    cell = P.Cell(P.CellConfig(Lx, Ly, d=d, D=D, chi=chi, p=p, n_si=2), torch.from_numpy(A).cuda())
    return cell, torch.from_numpy(np.concatenate(parts)).cuda()


def iterate(*case):
    """The state after one iteration from a random one, as a host array."""
    cell, state = prepare(*case)
    cell.set_state_device(state)
    cell.iterate("si")
    out = cell.get_state_device().cpu().numpy()
    cell.close()
    return out


def places(n, seed):
    return np.sort(np.random.default_rng(1000 + seed).choice(n, SAMPLES, replace=False))


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d-D%d-chi%d-seed%d" % (c[0], c[1], c[2], c[3], c[5]))
def test_state_of_wide_cuts(case):
    with np.load(GOLDEN) as f:
        want = f["_".join(map(str, case))]
    got = iterate(*case)
    rms = np.linalg.norm(got) / np.sqrt(got.size)
    got = got[places(got.size, case[5])]
    off = np.abs(got - want) / np.maximum(rms, np.abs(want))
    assert np.array_equal(got, want), off.max()


# the adjoint's forward pass makes the same rotations from k = 33 on; with others
# these four states differ by 4.4e-8 to 7.0e-8 of the rms
@pytest.mark.parametrize("seed", [4, 31, 36, 39])
def test_state_of_the_adjoint(seed):
    case = (2, 2, 2, 64, 6, seed)
    cell, state = prepare(*case)
    out = cell.move_vjp(state)[0].cpu().numpy()
    cell.close()
    want = iterate(*case)
    rms = np.linalg.norm(want) / np.sqrt(want.size)
    assert np.max(np.abs(out - want) / np.maximum(rms, np.abs(want))) <= 4e-8
