"""The host path of a statistics query when memory runs out: no C++ exception leaves
the C entry, and the next query works. Runs on the CPU: the library's calls to the HIP
runtime and its allocations are answered by a small preloaded stand-in."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstdlib>
#include <new>
static int left = 0;  // allocations until one fails; 0: none fails
extern "C" {
void stand_in_fail(int n) { left = n; }
int hipLaunchKernel(const void*, ...) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
}
void* operator new(size_t n) {
  if (left > 0 && --left == 0) throw std::bad_alloc();
  return malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
"""

QUERY = r"""
import ctypes, sys
import paper_1310_5045_amd as ppf
stand_in, fail_at = ctypes.CDLL(sys.argv[1]), int(sys.argv[2])
L, h = ppf.lib(), ctypes.c_void_p()
p = ppf.params()
room = ctypes.create_string_buffer(ppf.workspace_bytes(p) + 256)
at = (ctypes.addressof(room) + 255) // 256 * 256
assert L.ppf_create(ctypes.byref(p), ctypes.c_void_p(at), ppf.workspace_bytes(p), None,
                    ctypes.byref(h)) == ppf.PPF_OK
stand_in.stand_in_fail(fail_at)
first = L.ppf_sync(h)
stand_in.stand_in_fail(0)
assert first in (ppf.PPF_OK, ppf.PPF_ENOMEM), first
assert [L.ppf_sync(h) for _ in range(3)] == [ppf.PPF_OK] * 3
assert L.ppf_destroy(h) == ppf.PPF_OK
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("stand_in")
    (d / "s.cpp").write_text(STAND_IN)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(d / "s.so"), str(d / "s.cpp")],
                   check=True)
    return str(d / "s.so")


@pytest.mark.parametrize("fail_at", [0, 1, 2, 3])
def test_query_out_of_memory(stand_in, fail_at):
    preload = " ".join(os.environ.get("LD_PRELOAD", "").split() + [stand_in])
    r = subprocess.run([sys.executable, "-c", QUERY, stand_in, str(fail_at)], cwd=ROOT,
                       env=dict(os.environ, LD_PRELOAD=preload), capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
