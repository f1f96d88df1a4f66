"""Householder QR on every layout of its reduction tree: leaves of four and of eight
wavefronts, one to four levels, and nodes of 2, 3, 4, 5 and 8 children at the first
level and above it (2, 4 and 8 children are the register heights of the node kernel).
Which layout a shape takes is asked of the library, so that a change of the plan
cannot drop a branch here without notice.  The factorisation is checked as in
test_gpu_qr_edges.py, whose bound holds for any layout."""
import ctypes

import numpy as np
import pytest

import paper_2607_15158_amd as P
import synth as S

# N, k: leaves, of eight wavefronts, children of the last node of each level
LAYOUTS = [
    ((256, 100), (1, True, [])), ((300, 97), (1, True, [])), ((384, 192), (1, True, [])),
    ((385, 40), (3, False, [3])), ((385, 129), (2, False, [2])), ((640, 33), (5, False, [5])),
    ((1024, 48), (8, False, [8])), ((1153, 48), (4, True, [4])),
    ((3328, 32), (26, False, [2, 4])), ((3200, 17), (25, False, [1, 4])),
    ((8192, 33), (64, False, [8, 8])), ((9984, 32), (26, True, [2, 4])), ((13000, 40), (34, True, [2, 5])),
    ((24577, 8), (192, False, [8, 8, 3])), ((65664, 8), (171, True, [3, 6, 3])),
    ((524416, 3), (1366, True, [6, 3, 6, 3])),
]


def children(leaves):
    out = []
    while leaves > 1:
        out.append((leaves - 1) % 8 + 1)
        leaves = -(-leaves // 8)
    return out


@pytest.mark.parametrize("shape,layout", LAYOUTS, ids=lambda x: "-".join(map(str, x)) if isinstance(x[0], int) else None)
def test_layout(shape, layout):
    f = P._lib["_ZN5sictm14qr_plan_layoutEiiPiS0_S0_"]
    got = [ctypes.c_int(0) for _ in range(3)]
    f(*shape, *(ctypes.byref(x) for x in got))
    leaves, wide, levels = (x.value for x in got)
    assert (leaves, bool(wide), children(leaves)) == layout
    assert levels == len(layout[2])


@pytest.mark.gpu
@pytest.mark.parametrize("N,k", [s for s, _ in LAYOUTS])
def test_qr(N, k):
    torch = pytest.importorskip("torch")
    w = S.gaussian_block(N, k, 60)
    W = [w, w * np.logspace(0, -10, k), w.copy()]
    W[2][:, k // 2] = 0.0
    D = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in W]
    ok = P._lib["_ZN5sictm10qr_plan_okEii"]
    ok.restype = ctypes.c_bool
    if not ok(N, k):   # two leaves of 193 rows: refused, since a leaf holds 192
        assert (N, k) == (385, 129)
        with pytest.raises(P.CtmError):
            P.qr_f64(D)
        return
    P.qr_f64(D)
    u = 2.0 ** -53
    tol = 8 * np.sqrt(N) * k * u + 16 * u
    for w, d in zip(W, D):
        q = d.cpu().numpy()
        assert np.all(np.isfinite(q))
        assert np.linalg.norm(q.T @ q - np.eye(k)) <= tol
        r, nrm = q.T @ w, np.linalg.norm(w)
        assert np.linalg.norm(np.tril(r, -1)) <= tol * nrm
        assert np.all(np.diag(r) >= -tol * nrm)
        assert np.linalg.norm(q @ r - w) <= tol * nrm
