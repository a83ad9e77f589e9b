"""A dual mesh whose copy to the device fails reports it, and the next call
copies again instead of launching on memory that holds no W.  On the host: a
preloaded stand-in for the HIP calls that the upload makes fails the copy or
the synchronisation a given number of times and writes down what was called."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <cstdio>
#include <cstdlib>
static int env(const char *n) { const char *v = getenv(n); return v ? atoi(v) : 0; }
static int copies = env("FAIL_COPIES"), syncs = env("FAIL_SYNCS");
extern "C" {
int hipMalloc(void **p, size_t n) { *p = malloc(n); puts("malloc"); return 0; }
int hipFree(void *p) { free(p); puts("free"); return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { puts("copy"); return copies-- > 0 ? 1 : 0; }
int hipStreamSynchronize(void *) { puts("sync"); return syncs-- > 0 ? 1 : 0; }
struct dim3 { unsigned x, y, z; };
int __hipPushCallConfiguration(dim3, dim3, size_t, void *) { return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, void **s) { *g = *b = {1, 1, 1}; *n = 0; *s = 0; return 0; }
int hipLaunchKernel(const void *, dim3, dim3, void **, size_t, void *) { puts("launch"); return 0; }
int hipGetLastError() { return 0; }
}
"""

USER = """
import ctypes, sys
import numpy as np
from paper_2609_25653_amd import _lib
L = _lib.lib()
tri = np.array([[0, 1, 2]], np.int32)
h = ctypes.c_void_p()
assert L.ipc_dualmesh_create(tri.ctypes.data_as(_lib._I), 1, 3, 1, None, ctypes.byref(h)) == 0
for _ in range(3):
    print("apply", L.ipc_dualmesh_apply(h, ctypes.c_void_p(8), ctypes.c_void_p(8), 1), flush=True)
L.ipc_dualmesh_destroy(h)
print("end", flush=True)
"""


def _run(tmp_path, **fail):
    src, so = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(src), "-o", str(so)], check=True)
    pre = os.environ.get("LD_PRELOAD", "")
    env = dict(os.environ, LD_PRELOAD=f"{so}:{pre}" if pre else str(so), PYTHONPATH=ROOT, **{k: str(v) for k, v in fail.items()})
    out = subprocess.run(["stdbuf", "-o0", sys.executable, "-c", USER], env=env, capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    return out.stdout.split("\n")


@pytest.mark.parametrize("fail", [dict(), dict(FAIL_COPIES=1), dict(FAIL_SYNCS=1), dict(FAIL_COPIES=1, FAIL_SYNCS=1)])
def test_a_failed_upload_is_made_again(fail, tmp_path):
    from paper_2609_25653_amd import _lib
    if not os.path.exists(_lib.SO_PATH):
        pytest.skip("library not built")
    calls = [c for c in _run(tmp_path, **fail) if c]
    assert calls[-1] == "end"
    held = False           # the oracle: a W that was copied and synchronised without an error, and is not freed
    live = launches = 0
    bad = sum(fail.values())
    for k, c in enumerate(calls):
        if c == "malloc":
            live += 1
        elif c == "free":
            live -= 1
            held = False
        elif c == "sync":
            held = calls[k + 1] == "launch"
        elif c == "launch":
            assert held, calls
            launches += 1
    assert launches == 3 - bad and live == 0
    assert [c for c in calls if c.startswith("apply")] == ["apply 7" if k < bad else "apply 0" for k in range(3)]   # 7: IPC_E_DEVICE
