"""Runs Python code against libdd.so on the host-only HIP runtime of fake_hip.cpp,
in a process of its own.  The code finds `lib` (the library's C functions), `dd`
(the package), `np`, `C` (ctypes), `fake` (the runtime's test functions), `scan`
(a handle from Scan's arguments) and `launches(clear=True)`, a list of (kernel,
blocks in x, blocks in y)."""
import os
import pathlib
import shutil
import subprocess
import sys

import pytest

HERE = pathlib.Path(__file__).resolve().parent
ROOT = HERE.parent

PRELUDE = r"""
import ctypes as C, os, re, sys
sys.path.insert(0, os.environ["FAKE_ROOT"])
import numpy as np
import paper_2507_00294_amd as dd
fake = C.CDLL(os.environ["FAKE_HIP"])
fake.fake_log.restype = C.c_char_p
fake.fake_peak.restype = C.c_size_t
fake.fake_limit.argtypes = [C.c_size_t]
lib = dd.load_library()
def scan(*a, **k): return dd.Scan(*a, **k)
def launches(clear=True):
    out = []
    for line in fake.fake_log(1 if clear else 0).decode().splitlines():
        name, x, y = line.split()
        out.append((re.sub(r"^_ZN2dd(?:2nn|12_GLOBAL__N_1)*\d+", "", name), int(x), int(y)))
    return out
def ok(rc): assert rc == 0, (rc, lib.dd_last_error())
def buf(n): return np.zeros(int(n))
def ptr(a): return a.ctypes.data_as(C.c_void_p)
"""


def run(tmp_path, code):
    gxx = shutil.which("g++")
    if not gxx or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no g++ or HIP headers")
    if not (ROOT / "paper_2507_00294_amd/libdd.so").exists():
        pytest.skip("libdd.so is not built")
    so = tmp_path / "libfakehip.so"
    subprocess.run([gxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-w", str(HERE / "fake_hip.cpp"), "-o", str(so)],
                   check=True)
    env = dict(os.environ, FAKE_HIP=str(so), FAKE_ROOT=str(ROOT))
    env["LD_PRELOAD"] = ":".join(p for p in (os.environ.get("LD_PRELOAD", ""), str(so)) if p)
    r = subprocess.run([sys.executable, "-c", PRELUDE + code], env=env, cwd=tmp_path,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    return r.stdout
