"""What the library asks of the HIP runtime, seen by a small library with the
runtime's entry points that a child process loads before it."""
import json
import os
import subprocess
import sys

import pytest

import paper_1805_01450_amd as q
from paper_1805_01450_amd.build import hip_runtime_dir

pytestmark = pytest.mark.gpu

SHIM = r"""
#include <dlfcn.h>
#include <cstddef>
#include <map>
#include <mutex>
static void* of(const char* name) { return dlsym(dlopen(RUNTIME_DIR "/libamdhip64.so", RTLD_LAZY), name); }
static std::mutex mu;
static int n_host = 0, n_shrunk = 0, n_limits = 0;
static std::map<const void*, int> limit;
static unsigned long long ones = 0, zeros = 0;
extern "C" int host_allocations() { return n_host; }
extern "C" int limits_set() { return n_limits; }
extern "C" int limits_lowered() { return n_shrunk; }
extern "C" unsigned long long slice_ones() { return ones; }
extern "C" unsigned long long slice_zeros() { return zeros; }
extern "C" int hipHostMalloc(void** p, size_t n, unsigned flags) {
  ++n_host;
  static auto f = (int (*)(void**, size_t, unsigned))of("hipHostMalloc");
  return f(p, n, flags);
}
extern "C" int hipFuncSetAttribute(const void* fn, int attr, int value) {
  {
    std::lock_guard<std::mutex> lk(mu);
    ++n_limits;
    if (limit.count(fn) && value < limit[fn]) ++n_shrunk;
    limit[fn] = value;
  }
  static auto f = (int (*)(const void*, int, int))of("hipFuncSetAttribute");
  return f(fn, attr, value);
}
// a register kernel's launch: slices args[2] .. args[2] + args[1] - 1
extern "C" int hipModuleLaunchKernel(void* fn, unsigned gx, unsigned gy, unsigned gz, unsigned bx, unsigned by,
                                     unsigned bz, unsigned lds, void* stream, void** args, void** extra) {
  const unsigned long long n = *(unsigned long long*)args[1], first = *(unsigned long long*)args[2];
  for (unsigned long long s = first; s < first + n; ++s) ones |= s, zeros |= ~s;
  static auto f = (int (*)(void*, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, void*, void**,
                           void**))of("hipModuleLaunchKernel");
  return f(fn, gx, gy, gz, bx, by, bz, lds, stream, args, extra);
}
"""
HEAD = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.slice_ones.restype = shim.slice_zeros.restype = ctypes.c_ulonglong
import numpy as np
import paper_1805_01450_amd as q
from workload import generate_circuit, random_bitstrings
def plan(n, depth, k, **kw):
    c = q.Circuit(generate_circuit(n, depth, 0))
    sl, order = c.plan_slices(k_req=k, time_budget_s=1.0, flags=q.QGM_PLAN_DETERMINISTIC)
    return q.Plan(c, sl, order, **kw)
"""


def _child(tmp_path, code):
    src, lib = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", f'-DRUNTIME_DIR="{hip_runtime_dir()}"', str(src), "-o", str(lib),
                    "-ldl"], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(q.__file__)))
    r = subprocess.run([sys.executable, "-c", HEAD + code, str(lib)], cwd=root, capture_output=True, text=True,
                       timeout=110)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    print("[runtime]", r.stdout.splitlines()[-1], flush=True)
    return json.loads(r.stdout.splitlines()[-1])


def test_host_calls_allocate_nothing(tmp_path):
    """Host memory for small inputs and results is allocated with the plan's
    tables, not by the first call that uses it: a call may run while another
    thread captures a graph."""
    out = _child(tmp_path, r"""
p = plan(4, 10, 0)
p.workspace(4)
before = shim.host_allocations()
a = p.amplitudes(random_bitstrings(16, 4, 1))
print(json.dumps({"in_call": shim.host_allocations() - before, "at_upload": before, "finite": bool(np.isfinite(a).all())}))
""")
    assert out["finite"] and out["at_upload"] >= 1 and out["in_call"] == 0


def test_lds_limits_are_never_lowered(tmp_path):
    """Plans share the interpreter's kernels, so one plan's limit of dynamic
    LDS must not replace a higher one that another thread is about to use."""
    out = _child(tmp_path, r"""
# level kernels of more and of less LDS, and one wavefront per 64 items
big, small = (plan(n, d, k, engine=q.QGM_ENGINE_INTERPRETER) for n, d, k in ((6, 20, 6), (5, 20, 6)))
for p in (big, small, big):
    for n_bs in (1, 100, 1000):
        p.workspace(n_bs)
print(json.dumps({"set": shim.limits_set(), "lowered": shim.limits_lowered()}))
""")
    assert out["set"] > 0 and out["lowered"] == 0


def test_one_wavefront_form_is_compared_over_all_slice_bits(tmp_path):
    """The form is used where it gives the cut's bits; the slices it is
    compared on (the only launches here) have every slice bit at 0 and at 1."""
    out = _child(tmp_path, r"""
p = plan(6, 25, 10, prec=q.QGM_C64)
p.workspace(1)
every = (1 << p.k) - 1
print(json.dumps({"k": p.k, "ones": shim.slice_ones() & every, "zeros": shim.slice_zeros() & every}))
""")
    assert out["ones"] == out["zeros"] == (1 << out["k"]) - 1
