"""A launch that the runtime refuses is reported by the call that made it (run on
an MI355X).

A host library that stands before the HIP runtime refuses the n-th launch of
an augmented solve (the kernel is not launched and the runtime's error is set, as
for a launch that does not fit the device): for every n the call returns DEVICE,
whether its rounds stop at a check or at the iterate before it. The launches'
inputs are those of an ordinary solve; a refused one leaves its outputs as they
were. In a process of its own, since the library has to be loaded first.
"""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

REFUSE = r"""
#include <dlfcn.h>
struct dim3_ { unsigned x, y, z; };
static int left_ = -1, pending = 0, seen = 0;
static const int refused = 9;  // hipErrorInvalidConfiguration
static void* real(const char* name) {
    static void* h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    return dlsym(h, name);
}
extern "C" {
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, unsigned long lds, void* stream) {
    using F = int (*)(const void*, dim3_, dim3_, void**, unsigned long, void*);
    static F fn = (F)real("hipLaunchKernel");
    seen++;
    if (left_ >= 0 && left_-- == 0) return pending = refused;
    return fn(f, g, b, args, lds, stream);
}
int hipGetLastError() {
    using F = int (*)();
    static F fn = (F)real("hipGetLastError");
    const int e = fn(), p = pending;
    pending = 0;
    return p ? p : e;
}
void refuse_arm(int n) { left_ = n; pending = seen = 0; }
int refuse_seen() { return seen; }
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
import torch
import kktgen
from paper_2403_15913_amd import kkt
dev = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")
pat = kktgen.nmpc_pattern(6, 5, 2)
v = kktgen.nmpc_values(pat, kktgen.rng_for(13, 1), 1e-3, 1e3)
r1, r2, r4 = dev(v.b), dev(np.linspace(-1, 1, pat.m)), dev(np.linspace(1, 2, pat.m))
vals = [dev(a) for a in (v.w_vals, v.j_vals, v.sigma_x, v.sigma_s)]
f = kkt.Factor(kkt.Symbolic.from_pattern(pat))
f.keep_augmented(True)
def solve(n, tol):
    f.refactor(*vals)
    assert f.status()[0] == 0
    x, ds, dz = (torch.zeros(k, dtype=torch.float64, device="cuda") for k in (pat.n, pat.m, pat.m))
    torch.cuda.synchronize()
    shim.refuse_arm(n)
    try:
        code = f.solve_augmented(r1, r2, r4, x, ds, dz, tol=tol)["status"]
    except kkt.KKTError as e:
        code = e.status
    seen = shim.refuse_seen()
    shim.refuse_arm(-1)
    torch.cuda.synchronize()
    return code, seen
# tol 1e-14 stops at a check; tol 0 stops where the error no longer halves
for tol, want in ((1e-14, 0), (0.0, 6)):
    code, total = solve(-1, tol)
    assert code == want and total > 10, (tol, code, total)
    silent = [n for n in range(total) if solve(n, tol)[0] != 10]
    print(f"tol {tol}: {total} launches, not reported: {silent}", flush=True)
    assert not silent, (tol, silent)
    assert solve(-1, tol)[0] == want
"""


def test_refused_launches_are_reported(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, so, child = tmp_path / "refuse.cpp", tmp_path / "librefuse.so", tmp_path / "child.py"
    src.write_text(REFUSE)
    child.write_text(CHILD)
    subprocess.run([gxx, "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    r = subprocess.run([sys.executable, str(child), str(so), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
