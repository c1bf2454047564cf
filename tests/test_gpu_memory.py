"""Calls that cannot have the memory they would like: the objective and the
adjoint take the schedules that keep fewer fields, with the same bits, and fail
with SWEPT_ENOMEM only where those do not fit either.  A small library whose
hipMalloc refuses sizes above a limit stands in for a full GPU; it is loaded
ahead of the HIP runtime in a process of its own."""
import os
import subprocess
import sys

import pytest

from tests.conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
typedef int (*alloc_t)(void**, size_t);
static alloc_t real;
static size_t limit = (size_t)-1;
static int refused;
void shim_real(alloc_t f) { real = f; }
void shim_limit(size_t bytes) { limit = bytes; refused = 0; }
int shim_refused(void) { return refused; }
int hipMalloc(void** p, size_t bytes)
{
    if (bytes > limit) {
        ++refused;
        return 2;   /* hipErrorOutOfMemory */
    }
    return real(p, bytes);
}
"""

SCRIPT = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_limit.argtypes = [ctypes.c_size_t]
sys.path.insert(0, sys.argv[2])
import torch
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64.so" in l)
shim.shim_real(ctypes.cast(ctypes.CDLL(path).hipMalloc, ctypes.c_void_p))
import workloads
import paper_1504_01380_amd as sw
sw.init(0)

MIB = 1 << 20
n = 1 << 16
PAR = {"heat": [0.3], "ks": [workloads.KS_DT, workloads.KS_DX]}
u0 = torch.from_numpy(workloads.smoothed_noise(n, seed=1)).cuda()
cot = torch.from_numpy(workloads.white_noise(n, seed=2)).cuda()
room = [torch.empty_like(u0) for _ in range(12)]     # torch's pool has room for the results
del room
torch.cuda.synchronize()

def call(what, stencil, nsteps, first, limit):
    "the result on fresh scratch, and how many allocations were refused"
    sw.finalize()
    shim.shim_limit(limit)
    try:
        r = getattr(sw, what)(u0, nsteps, stencil, PAR[stencil], window_first=first,
                              window_weight=0.01, cot_final=cot)
        torch.cuda.synchronize()
        return r, shim.shim_refused()
    finally:
        shim.shim_limit(2 ** 64 - 1)

def same(a, b):
    return bool((a.view(torch.int64) == b.view(torch.int64)).all())

for stencil in ("heat", "ks"):
    want, none = call("objective", stencil, 200, 0, 2 ** 64 - 1)
    got, refused = call("objective", stencil, 200, 0, 8 * MIB)
    assert none == 0 and refused == 1 and same(want, got), (stencil, refused)
    # 200 fields of 0.5 MiB; the swept adjoint's edges: heat 8 MiB, KS 84
    want, none = call("adjoint", stencil, 200, 0, 2 ** 64 - 1)
    got, refused = call("adjoint", stencil, 200, 0, (32 if stencil == "heat" else 92) * MIB)
    assert none == 0 and refused == 1 and same(want, got), (stencil, refused)
    for what in ("objective", "adjoint"):
        try:
            call(what, stencil, 200, 0, 64 << 10)
            raise SystemExit("no error")
        except sw.SweptError as e:
            assert e.code == -3, e        # SWEPT_ENOMEM
    got, none = call("adjoint", stencil, 200, 0, 2 ** 64 - 1)
    assert none == 0 and same(want, got)  # and the next call is served again
    print(stencil, "ok", flush=True)

# heat keeps up to 4 GiB (8192 fields of 0.5 MiB), and beyond that takes the
# swept adjoint without asking for more
want, refused = call("adjoint", "heat", 8192, 1, 1024 * MIB)
assert refused == 1, refused
got, refused = call("adjoint", "heat", 8193, 1, 1024 * MIB)
assert refused == 0, refused
print("switch ok", flush=True)
"""


def test_fallbacks_without_memory(tmp_path):
    src, lib = tmp_path / "shim.c", tmp_path / "libshim.so"
    src.write_text(SHIM)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib)])
    r = subprocess.run([sys.executable, "-u", "-c", SCRIPT, str(lib), ROOT], cwd=ROOT, timeout=100,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0 and r.stdout.endswith("switch ok\n"), r.stdout[-3000:]
