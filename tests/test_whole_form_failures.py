"""The one-wavefront form of a cut register plan is an addition: where it
cannot be made or loaded, the plan runs its cut.

A small library with the runtime's entry points, loaded into a child process
before the runtime, lets a chosen call fail."""
import json
import os
import subprocess
import sys

import pytest

import paper_1805_01450_amd as q
from paper_1805_01450_amd.build import hip_runtime_dir

SHIM = r"""
#include <dlfcn.h>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
static std::atomic<int> n_compiles{0}, n_loads{0};
static void* of(const char* lib, const char* name) {
  return dlsym(dlopen((std::string(RUNTIME_DIR "/") + lib).c_str(), RTLD_LAZY), name);
}
static bool fails(const char* what) { return std::strcmp(std::getenv("FAIL"), what) == 0; }
extern "C" int compiles() { return n_compiles; }
extern "C" int loads() { return n_loads; }
extern "C" int hiprtcCreateProgram(void** p, const char* src, const char* name, int n, const char** h, const char** i) {
  ++n_compiles;
  if (fails(std::strstr(src, "int never = 0") ? "form" : "cut")) throw std::bad_alloc();
  static auto f = (int (*)(void**, const char*, const char*, int, const char**, const char**))of("libhiprtc.so", "hiprtcCreateProgram");
  return f(p, src, name, n, h, i);
}
extern "C" int hipModuleLoadData(void** m, const void* image) {
  if (++n_loads > 1 && fails("load")) return 301;
  static auto f = (int (*)(void**, const void*))of("libamdhip64.so", "hipModuleLoadData");
  return f(m, image);
}
"""
CHILD = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_1805_01450_amd as q
from workload import generate_circuit, random_bitstrings
c = q.Circuit(generate_circuit(6, 25, 0))
sl, order = c.plan_slices(k_req=10, time_budget_s=1.0, flags=q.QGM_PLAN_DETERMINISTIC)
try:
    p = q.Plan(c, sl, order, prec=q.QGM_C64)
except q.QgmError as e:
    print(json.dumps({"status": e.status}), flush=True)
    sys.exit(0)
out = {"waves": p.stats()["waves"], "compiles": shim.compiles()}
if sys.argv[2] == "run":
    bits = random_bitstrings(36, 400, 21)
    large, small = p.amplitudes(bits), p.amplitudes(bits[:2])
    out.update(compiles=shim.compiles(), loads=shim.loads(), finite=bool(np.isfinite(large).all()),
               same=bool((large[:2] == small).all()))
print(json.dumps(out), flush=True)
"""


def _child(tmp_path, fail, what):
    src, lib = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", f'-DRUNTIME_DIR="{hip_runtime_dir()}"', str(src), "-o", str(lib),
                    "-ldl"], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(q.__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib), what], cwd=root, capture_output=True, text=True,
                       timeout=110, env=dict(os.environ, FAIL=fail))
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return json.loads(r.stdout.splitlines()[-1])


def test_exceptions_of_the_two_compiles(tmp_path):
    """The two kernels compile side by side.  One that throws in the form's
    leaves the cut; one in the cut's waits for the other and comes back as a
    status; neither ends the process."""
    assert _child(tmp_path, "form", "create") == {"waves": 4, "compiles": 2}
    assert _child(tmp_path, "cut", "create")["status"] != 0


@pytest.mark.gpu
@pytest.mark.parametrize("fail", ["load"])
def test_plan_without_the_form_runs_its_cut(fail, tmp_path):
    print("[whole-form] failing", fail, flush=True)
    out = _child(tmp_path, fail, "run")
    print(out, flush=True)
    assert out["waves"] > 1 and out["finite"] and out["same"]
    assert out["loads"] == 2  # the form's was asked for, and refused
