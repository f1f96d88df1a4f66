"""The QR workspace of N rows holds every QR of fewer rows: contexts and cells carve
it for their full size and run it on smaller environments too (growth moves, the
correlation length).  Host function only, no GPU."""
import ctypes

import pytest

import paper_2607_15158_amd as P


@pytest.mark.parametrize("k", [1, 8, 31, 32, 33, 64, 97, 128, 136, 160, 192])
def test_workspace_never_shrinks_with_more_rows(k):
    size = P._lib["_ZN5sictm18qr_workspace_bytesEiii"]
    size.restype, size.argtypes = ctypes.c_size_t, [ctypes.c_int] * 3
    ok = P._lib["_ZN5sictm10qr_plan_okEii"]
    ok.restype, ok.argtypes = ctypes.c_bool, [ctypes.c_int] * 2
    most, at = 0, 0
    for n in list(range(k, 4000)) + list(range(8000, 8700)) + [24000, 24576, 24577, 70000, 746496]:
        if not ok(n, k):
            continue
        b = size(8, n, k)
        assert b >= most, (n, at)
        most, at = b, n
