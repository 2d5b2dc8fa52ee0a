"""The library's host code against a stand-in for the HIP runtime that tracks
streams, events, captures and graphs (host_runtime.cpp): no call may destroy
a graph that can still be running, leave a capture unjoined, work while
another device is current or launch beyond the documented limits.  Kernels do nothing, so outputs are not looked at."""
import os
import re
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
BINDING = os.path.join(HERE, os.pardir, "paper_2403_08148_amd", "_binding.py")

DRIVER = r'''
import ctypes as C, importlib.util, random, sys
import numpy as np
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # (the library's runtime by its soname)
spec = importlib.util.spec_from_file_location("binding", sys.argv[2])
B = importlib.util.module_from_spec(spec)
spec.loader.exec_module(B)
L = B.load()

def dptr(x):
    return x.ctypes.data_as(C.POINTER(C.c_double))

def run(calls, n, fp64, rng):
    nb = (C.c_int32 * 1)(n)
    h = C.c_void_p()
    info = B.gcme_create_info(1, C.cast(nb, C.POINTER(C.c_int32)), B.GCME_FP64 if fp64 else B.GCME_MIXED, 0, None, 1)
    assert L.gcme_create(C.byref(info), C.byref(h)) == 0
    box = max(4.2, (n / 2.5) ** (1 / 3))
    keep = []
    def ok(st):
        assert st == 0, (st, L.gcme_last_error(h))
    def params(dt=0.02, s=0.5):
        A, sg, a = np.full(4, 25.0), np.full(2, s), np.array([0.4, 0.6])
        keep.append((A, sg, a))
        p = B.gcme_params((C.c_double * 3)(box, box, box), 2.0, 1.1, (C.c_int32 * 3)(24, 24, 24), 5, 1.0, 2, dptr(A), dptr(sg),
                          dptr(a), None, 1.0, dt, 1.0, 0, 0.0, 0.0, 0.0)
        ok(L.gcme_set_params(h, 0, C.byref(p)))
    pos, vel, F = np.random.default_rng(n).random((3, 3 * n))
    E, V = np.zeros(B.GCME_N_TERMS), np.zeros(6)
    typ, z = np.arange(n, dtype=np.int32) % 2, np.zeros(n, dtype=np.int32)
    z[:n // 8 * 2] = np.tile([1, -1], n // 8)
    def state():
        ok(L.gcme_set_state(h, pos.ctypes.data, vel.ctypes.data, typ.ctypes.data, z.ctypes.data))
    def evaluate():
        io = B.gcme_io()
        io.pos, io.force, io.energy = pos.ctypes.data, F.ctypes.data, E.ctypes.data
        ok(L.gcme_forces_energy(h, C.byref(io)))
    def observed(k):
        io = B.gcme_io()
        io.energy, io.virial = E.ctypes.data, V.ctypes.data
        ok(L.gcme_step(h, k, C.byref(io)))
    def tune(**kw):
        t = B.gcme_tuning(*[kw.get(f, -1) for f, _ in B.gcme_tuning._fields_])
        ok(L.gcme_set_tuning(h, C.byref(t)))
    do = {"state": state, "evaluate": evaluate, "step": lambda: ok(L.gcme_step(h, rng.randint(0, 30), None)),
          "observed": lambda: observed(rng.randint(1, 3)), "pairs": lambda: params(s=rng.uniform(0.4, 0.6)),
          "params": lambda: params(dt=rng.choice([0.01, 0.02])), "layout": lambda: tune(stream_layout=rng.randint(0, 5)),
          "cells": lambda: tune(cells_per_cutoff=rng.randint(1, 4)),
          "clusters": lambda: tune(beads_per_cluster=rng.choice([2, 4, 8]), charges_per_cluster=rng.choice([2, 4, 8])),
          "lists": lambda: tune(direct_pairs=rng.randint(0, 3)), "sync": lambda: ok(L.gcme_sync(h)),
          "get": lambda: ok(L.gcme_get_state(h, pos.ctypes.data, vel.ctypes.data, None)),
          "autotune": lambda: ok(L.gcme_autotune(h)),
          "stages": lambda: ok(L.gcme_time_stages(h, 2, (C.c_double * B.GCME_N_STAGES)())),
          "profile": lambda: ok(L.gcme_profile_step(h, 2, (C.c_double * B.GCME_N_STAGES)()))}
    params()
    state()
    for c in calls or rng.choices(sorted(set(do) - {"autotune"}), k=25):
        stub.hipSetDevice(1)  # (a program's own choice between two calls)
        do[c]()
    L.gcme_destroy(h)

rng = random.Random(5)
calls = sys.argv[3].split()
for n in (40, 700, 1023, 4097, 9000):
    for fp64 in (False, True):
        print("case", n, fp64, calls, flush=True)
        run(calls, n, fp64, rng)
sys.exit(1 if stub.stub_misuses() else 0)
'''


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    lib = os.path.join(os.path.dirname(BINDING), "libgcme.so")
    if not os.path.exists(lib) or not shutil.which("g++"):
        pytest.skip("library not built, or no compiler")
    soname = re.search(rb"libamdhip64\.so\.\d+", open(lib, "rb").read()).group().decode()
    out = str(tmp_path_factory.mktemp("rt") / soname)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-Wl,-soname,{soname}",
                           os.path.join(HERE, "host_runtime.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("calls", ["step layout step", "observed layout observed", "step clusters step", "step cells step",
                                   "step params step", "step pairs step", "step state step", "step stages profile step",
                                   "step autotune step", ""], ids=lambda c: c.replace(" ", "-") or "any")
def test_no_misuse_of_the_runtime(runtime, calls):
    r = subprocess.run([sys.executable, "-c", DRIVER, runtime, BINDING, calls], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
