"""What a context does on a device that is nearly full: the library, linked to a program that brings its own allocator (host memory with
a limit) and device queries, creates its contexts without a GPU."""
import os
import subprocess

import pytest

from paper_2504_18154_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "ecoserve.h"
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
static size_t room = 0, held = 0;
extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { return std::memset(p, 0, sizeof *p), p->multiProcessorCount = 256, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (n > room - held) return hipErrorOutOfMemory;
  size_t* const m = static_cast<size_t*>(std::malloc(n + 256));
  m[0] = n;
  held += n;
  *p = m + 32;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (p) {
    size_t* const m = static_cast<size_t*>(p) - 32;
    held -= m[0];
    std::free(m);
  }
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
}
int main() {
  ecoserve_layout lay = {};
  lay.num_q_heads = 40, lay.num_kv_heads = 8, lay.head_dim = 128, lay.block_size = 16, lay.num_blocks = 4096, lay.dtype = ECOSERVE_BF16;
  size_t bytes[3];
  int st[3], i = 0;
  for (size_t mb : {1024, 40, 0}) {  // all of it, all but the pieces' 65 MiB, nothing
    room = mb << 20;
    ecoserve_ctx* c = nullptr;
    st[i] = ecoserve_create(&c, 0, &lay, 64, 256);
    bytes[i] = ecoserve_workspace_bytes(c);
    if ((st[i] == ECOSERVE_OK) != (c != nullptr) || bytes[i] != held) return std::printf("%zu MiB: status %d, %zu bytes, held %zu\n", mb, st[i], bytes[i], held), 1;
    if (c) ecoserve_destroy(c);
    if (held) return std::printf("%zu bytes kept\n", held), 1;
    ++i;
  }
  std::printf("%d %d %d %zu\n", st[0], st[1], st[2], (bytes[0] - bytes[1]) >> 20);
}
"""


def test_a_nearly_full_device_does_without_the_prefill_pieces(tmp_path):
    if not os.path.exists(build.LIB):
        pytest.skip("the library is not built")
    src, exe = tmp_path / "full.cpp", tmp_path / "full"
    src.write_text(PROGRAM)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build._hipcc())))
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.INCLUDE, "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe), "-rdynamic", build.LIB,
                    f"-Wl,-rpath,{os.path.dirname(build.LIB)}:{os.path.join(rocm, 'lib')}", f"-Wl,-rpath-link,{os.path.join(rocm, 'lib')}"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.split() == ["0", "0", "3", "65"], r.stdout + r.stderr[-500:]
