"""Runs a Python snippet against libfrdvm with tests/hip_stub.c in place of
the HIP runtime (no GPU needed), in a process of its own.  The snippet finds
``F`` (the binding), ``W`` (workloads), ``np``, ``C`` (ctypes) and ``hip``
(the stub's controls); it reports through ``print``."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
hip = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
hip.stub_find.restype, hip.stub_find.argtypes = C.c_void_p, [C.c_size_t, C.c_int]
hip.stub_live.restype = C.c_size_t
hip.stub_allocs.restype = hip.stub_launches.restype = C.c_long
hip.stub_fail_at.argtypes = [C.c_long]
hip.stub_capacity.argtypes = [C.c_size_t]
import numpy as np
import workloads as W
from paper_2312_06567_amd import frdvm as F
"""


def run(tmp_path, code, env=None):
    so = str(tmp_path / "libhipstub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "hip_stub.c")], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + code], capture_output=True, text=True,
                       timeout=300, env={**os.environ, **(env or {})})
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
