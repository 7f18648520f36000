"""What a context does on a device that is nearly full: the library, linked to a program that brings its own allocator (host memory with
a limit) and device queries, creates its contexts without a GPU."""
import os
import subprocess

import pytest

from paper_2504_18154_amd import build

ALLOCATOR = r"""
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
"""

PROGRAM = r"""
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


PLAIN = r"""
int main() {
  ecoserve_layout lay = {};
  lay.num_q_heads = 32, lay.num_kv_heads = 8, lay.head_dim = 64, lay.block_size = 16, lay.num_blocks = 4096, lay.dtype = ECOSERVE_BF16;
  const size_t plain = (size_t)256 * 32 * (8192 / 64 + 2) * 66 * 4;  // the plain kernels' states
  room = (size_t)1 << 30;
  ecoserve_ctx* c = nullptr;
  if (ecoserve_create(&c, 0, &lay, 256, 512)) return std::printf("not created\n"), 1;
  const size_t made = held;
  if (made > plain / 4) return std::printf("%zu bytes without the plain kernels, their states are %zu\n", made, plain), 1;
  room = made;  // (nothing left: the option is refused and the context is as it was)
  if (ecoserve_set_option(c, ECOSERVE_OPT_FORCE_PLAIN, 1) != ECOSERVE_ENOMEM || ecoserve_workspace_bytes(c) != held || held != made) return std::printf("no room: %zu of %zu\n", held, made), 1;
  if (ecoserve_set_option(c, ECOSERVE_OPT_DECODE_SPLIT_TOKENS, 64) != ECOSERVE_ENOMEM || ecoserve_workspace_bytes(c) != held || held != made) return std::printf("no room: %zu of %zu\n", held, made), 1;
  room = (size_t)1 << 30;
  for (int on : {1, 0, 1})
    if (ecoserve_set_option(c, ECOSERVE_OPT_FORCE_PLAIN, on) || held != made + plain || ecoserve_workspace_bytes(c) != held) return std::printf("plain %d: %zu of %zu + %zu\n", on, held, made, plain), 1;
  size_t forced = 0;
  for (int tokens : {1024, 64, 0, 4096}) {  // (states for any length of slices, once)
    if (ecoserve_set_option(c, ECOSERVE_OPT_DECODE_SPLIT_TOKENS, tokens) || ecoserve_workspace_bytes(c) != held || (forced && held != forced)) return std::printf("slices of %d: %zu of %zu\n", tokens, held, forced), 1;
    forced = held;
  }
  ecoserve_destroy(c);
  // (bf16, 128): an option that is refused leaves the states that there were
  lay.head_dim = 128;
  if (held || ecoserve_create(&c, 0, &lay, 256, 512)) return std::printf("not created\n"), 1;
  const size_t tuned = room = held;
  if (ecoserve_set_option(c, ECOSERVE_OPT_FORCE_PLAIN, 1) != ECOSERVE_ENOMEM || ecoserve_workspace_bytes(c) != tuned || held != tuned) return std::printf("no room: %zu of %zu\n", held, tuned), 1;
  ecoserve_destroy(c);
  std::printf("%zu\n", held);
}
"""


def _run(tmp_path, program):
    if not os.path.exists(build.LIB):
        pytest.skip("the library is not built")
    src, exe = tmp_path / "full.cpp", tmp_path / "full"
    src.write_text(ALLOCATOR + program)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build._hipcc())))
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.INCLUDE, "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe), "-rdynamic", build.LIB,
                    f"-Wl,-rpath,{os.path.dirname(build.LIB)}:{os.path.join(rocm, 'lib')}", f"-Wl,-rpath-link,{os.path.join(rocm, 'lib')}"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr[-500:]
    return r.stdout.split()


def test_a_nearly_full_device_does_without_the_prefill_pieces(tmp_path):
    assert _run(tmp_path, PROGRAM) == ["0", "0", "3", "65"]


def test_states_of_the_plain_kernels_come_with_the_option(tmp_path):
    """A layout other than (bf16, 128): what only ECOSERVE_OPT_FORCE_PLAIN or a forced length of slices use is not there before, comes once, and a device
    without room for it refuses the option, of any layout, and the context is as it was."""
    assert _run(tmp_path, PLAIN) == ["0"]
