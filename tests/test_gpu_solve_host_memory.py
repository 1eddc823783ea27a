"""A solve takes no host memory of its own (run on an MI355X): everything is
allocated with the factor or the batch, so a solve cannot fail, or throw out of
the C interface, for want of it.

A host library that stands before the C++ runtime counts the allocations whose
caller is libkkt, during the first solve of a factor (with and without a report,
in the workspace form) and of a batch. In a process of its own, since the library
has to be loaded first.
"""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNT = r"""
#include <dlfcn.h>
#include <stdlib.h>
#include <string.h>
#include <new>
static bool on = false;
static int counted = 0;
void* operator new(size_t n) {
    if (on) {
        on = false;
        Dl_info d;
        if (dladdr(__builtin_return_address(0), &d) && d.dli_fname && strstr(d.dli_fname, "libkkt.so")) counted++;
        on = true;
    }
    void* p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
extern "C" void count_start() { counted = 0; on = true; }
extern "C" int count_stop() { on = false; return counted; }
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
v = kktgen.nmpc_values(pat, kktgen.rng_for(14, 1), 1e-2, 1e2)
vals = [dev(a) for a in (v.w_vals, v.j_vals, v.sigma_x, v.sigma_s)]
shim.count_start()
sym = kkt.Symbolic.from_pattern(pat)
assert shim.count_stop() > 0, "the analysis allocates: the counter must see it"
def count(solve, b, x):
    torch.cuda.synchronize()
    shim.count_start()
    solve(b, x)
    return shim.count_stop()
got = {}
for name, call in (("report", lambda f: f.solve), ("queued", lambda f: lambda b, x: f.solve(b, x, info=False)),
                   ("workspace", lambda f: f.solve_noalloc)):
    f = kkt.Factor(sym)
    f.refactor(*vals)
    got[name] = count(call(f), dev(v.b), torch.zeros(pat.n, dtype=torch.float64, device="cuda"))
B = kkt.Batch([sym] * 3)
B.refactor(*[torch.cat([a] * 3) for a in vals])
got["batch"] = count(B.solve, torch.cat([dev(v.b)] * 3), torch.zeros(3 * pat.n, dtype=torch.float64, device="cuda"))
print(got, flush=True)
assert not any(got.values()), got
"""


def test_solves_allocate_no_host_memory(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, so, child = tmp_path / "count.cpp", tmp_path / "libcount.so", tmp_path / "child.py"
    src.write_text(COUNT)
    child.write_text(CHILD)
    subprocess.run([gxx, "-std=c++17", "-O1", "-fno-inline", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"],
                   check=True)
    r = subprocess.run([sys.executable, str(child), str(so), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
