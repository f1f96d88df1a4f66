"""State vectors go to the device by one kernel only where that kernel can reach
them: on the current device, in one allocation, and where the context's own
buffers are on that device too (a kernel on the context's stream has no access to
another device's memory; a copy has).  The runtime's answers are played by a small
library that is loaded before it, so no GPU is needed."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_15158_amd", "libsictm.so")

# device 0 owns 1 MiB at 16 MiB, device 1 at 32 MiB, the host 1 MiB at 48 MiB
PLAY = r"""
#include <hip/hip_runtime_api.h>
#include <cstdint>
static int current = 0;
static uintptr_t block(const void* p) { return (uintptr_t)p >> 24; }
extern "C" {
void play_device(int d) { current = d; }
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const uintptr_t b = block(p);
  if (b < 1 || b > 3) return hipErrorInvalidValue;
  *a = hipPointerAttribute_t{};
  a->type = b == 3 ? hipMemoryTypeHost : hipMemoryTypeDevice;
  a->device = b == 2 ? 1 : 0;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  *base = (hipDeviceptr_t)(block(p) << 24);
  *size = 1 << 20;
  return hipSuccess;
}
}
"""

ASK = r"""
import ctypes, sys
play = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
f = lib["_ZN5sictm17elem_device_rangeEPKvmS1_"]
f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
d0, d1, host, none = 1 << 24, 2 << 24, 3 << 24, 4 << 24
for cur, p, n, own, want in [
        (0, d0, 4096, d0 + 64, True), (1, d1, 4096, d1, True), (0, d0 + 64, (1 << 20) - 64, d0, True),
        (1, d1, 4096, d0, False), (0, d0, 4096, d1, False),      # the context on the other device
        (1, d0, 4096, d0, False), (0, d1, 4096, d0, False), (0, d1, 4096, d1, False),
        (0, d0 + 64, 1 << 20, d0, False),                        # past the allocation
        (0, host, 64, d0, False), (0, none, 64, d0, False), (0, d0, 64, host, False)]:
    play.play_device(cur)
    assert f(p, n, own) == want, (cur, hex(p), n, hex(own), want)
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="needs g++")
def test_packed_only_where_the_kernel_reaches(tmp_path):
    src, lib = tmp_path / "play.cpp", tmp_path / "libplay.so"
    src.write_text(PLAY)
    subprocess.run(["g++", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wl,-Bsymbolic",
                    str(src), "-o", str(lib)], check=True)
    subprocess.run([sys.executable, "-c", ASK, str(lib), LIB], check=True, timeout=120)
