"""What ctm_qr_f64 keeps between calls is bounded in bytes: workspaces of about 100
to 200 MB, in ascending size, push out the oldest, and both a destroyed context and
release_workspaces give back what is kept, measured as free memory of the device."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2607_15158_amd as P  # noqa: E402
import synth as S  # noqa: E402

MIB = 1 << 20
SLACK = 8 * MIB   # the allocator's granularity, for a handful of blocks
SHAPES = [(8, 6000, 160), (8, 8000, 160), (8, 10000, 160), (8, 12000, 160)]


def need(count, N, k):
    f = P._lib["_ZN5sictm18qr_workspace_bytesEiii"]
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int] * 3
    return f(count, N, k)


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def close(got, want):
    return want - SLACK <= got <= want + SLACK


def test_bytes_are_bounded_and_given_back():
    W = [torch.randn(SHAPES[-1][1] * 160, dtype=torch.float64, device="cuda") for _ in range(8)]
    ctx = P.Ctm(P.Config(d=2, D=2, chi=4, p=2, n_si=1),
                torch.from_numpy(S.product_plus_noise_site(2, 2, 3)).cuda())
    P.qr_f64([w[:64 * 16].view(64, 16) for w in W])   # the kernels' code is on the device
    P.release_workspaces()
    base = free()
    kept = []                                           # sizes, oldest first
    for c, N, k in SHAPES:
        n = need(c, N, k)
        assert 80 * MIB < n < 256 * MIB
        P.qr_f64([w[:N * k].view(N, k) for w in W])
        while sum(kept) + n > 256 * MIB:
            kept.pop(0)
        kept.append(n)
        assert close(base - free(), sum(kept)), (N, base - free(), kept)
    assert len(kept) < len(SHAPES)                      # some were pushed out
    before = free()
    ctx.close()                                         # its own memory is torch's
    assert close(free() - before, sum(kept)), (free() - before, kept)
    P.qr_f64([w[:6000 * 160].view(6000, 160) for w in W])
    before = free()
    P.release_workspaces()
    assert close(free() - before, need(*SHAPES[0]))
