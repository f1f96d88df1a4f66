"""The workspaces that ctm_qr_f64 and ctm_svd_f64 keep are given back: those of a
context's device when it is destroyed, whatever device is current then; those of the
current device by ctm_release_workspaces and when an allocation of the library fails
there, the serving arena's among them.  A small library that is loaded before the
runtime plays it (two devices of 1 GiB, kernels that do nothing), so no GPU is needed."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_15158_amd", "libsictm.so")

PLAY = r"""
#include <hip/hip_runtime_api.h>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
static int current = 0;
static size_t used[2];
static std::map<uintptr_t, std::pair<int, size_t>> blocks;
static uintptr_t next_at = (uintptr_t)1 << 40;
extern "C" {
void play_device(int d) { current = d; }
size_t play_used(int d) { return used[d]; }
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (used[current] + n > (size_t)1 << 30) return hipErrorOutOfMemory;
  used[current] += n;
  *p = (void*)next_at;
  blocks[next_at] = {current, n};
  next_at += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = blocks.find((uintptr_t)p);
  if (it == blocks.end()) return hipErrorInvalidValue;
  used[it->second.first] -= it->second.second;
  blocks.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)64; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)64; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToHost) memset(d, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { return hipMemcpyAsync(d, s, n, k, 0); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, hipStream_t) { return hipSuccess; }
}
"""

ASK = r"""
import ctypes, sys
play = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
play.play_used.restype = ctypes.c_size_t
lib = ctypes.CDLL(sys.argv[2])
V, I, Z, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t, ctypes.c_double
used = lambda: [play.play_used(d) for d in (0, 1)]


def qr(dev):
    play.play_device(dev)
    W = (V * 8)(*[(i + 1) << 32 for i in range(8)])
    assert lib.ctm_qr_f64(I(8), W, I(5184), I(160), None) == 0


class Config(ctypes.Structure):
    _fields_ = [("d", I), ("D", I), ("chi", I), ("p", I), ("n_si", I), ("proj", I), ("prec", I), ("stabilized", I),
                ("pinv_rtol", L), ("svd_driver", I), ("sym", I), ("recycle_sin2", L), ("min_si_moves", I), ("growth", I)]


def context(dev):
    play.play_device(dev)
    h, c = V(), Config(2, 2, 4, 2, 1, 1, 0, 1, 1e-12, 0, 0, 0.0, 3, 0)
    need = Z()
    assert lib.ctm_workspace_bytes(ctypes.byref(c), ctypes.byref(need)) == 0
    assert lib.ctm_init(ctypes.byref(h), ctypes.byref(c), V(1 << 32), None, V(1 << 36), need, None) == 0
    return h


lib.ctm_destroy.argtypes = [V]
lib.ctm_server_destroy.argtypes = [V]
qr(0)
qr(1)
block = used()[0]
assert block > 60 << 20 and used() == [block, block]
qr(0)
assert used() == [block, block]                      # the kept one
# a context of device 0 destroyed while device 1 is current
h = context(0)
play.play_device(1)
lib.ctm_destroy(h)
assert used() == [0, block], used()
# the current device's, by the call
qr(0)
play.play_device(1)
lib.ctm_release_workspaces()
assert used() == [block, 0], used()
# an arena that fits only without the kept block
play.play_device(0)
s = V()
lib.ctm_server_create.argtypes = [ctypes.POINTER(V), Z, I]
assert lib.ctm_server_create(ctypes.byref(s), (1 << 30) - (16 << 20), 4) == 0
assert used() == [(1 << 30) - (16 << 20), 0], used()
lib.ctm_server_destroy(s)
assert used() == [0, 0], used()
# what no block makes room for is refused as before
qr(0)
assert lib.ctm_server_create(ctypes.byref(s), 2 << 30, 4) != 0
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="needs g++")
def test_kept_blocks_are_given_back(tmp_path):
    src, lib = tmp_path / "play.cpp", tmp_path / "libplay.so"
    src.write_text(PLAY)
    subprocess.run(["g++", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wl,-Bsymbolic",
                    str(src), "-o", str(lib)], check=True)
    subprocess.run([sys.executable, "-c", ASK, str(lib), LIB], check=True, timeout=120)
