"""Runs the library's host side without a GPU, over native/fake_hip.c: device
memory is host memory, kernels do not run, allocations can fail.

As a module: ``run(script)`` builds the stand-in once per session and runs the
script in a process of its own, in which ``fake``, ``dbs``, ``lib`` and ``np``
are defined."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
_dir = None

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [{root!r}, {here!r}]
import numpy as np
import paper_2608_16308_amd as dbs
lib = dbs.lib()
def var(name, t=ctypes.c_long):
    return t.in_dll(fake, name)
"""


def build():
    global _dir
    if _dir is None:
        _dir = tempfile.TemporaryDirectory(prefix="fake_hip")
        d = _dir.name
        n = os.path.join(HERE, "native")
        subprocess.run(["gcc", "-O1", "-fPIC", "-c", os.path.join(n, "fake_hip.c"), "-o", d + "/a.o"], check=True)
        subprocess.run(["g++", "-O1", "-fPIC", "-I/opt/rocm/include", "-c", os.path.join(n, "fake_hip_layout.cpp"),
                        "-o", d + "/b.o"], check=True)
        subprocess.run(["g++", "-shared", "-o", d + "/libfakehip.so", d + "/a.o", d + "/b.o"], check=True)
    return os.path.join(_dir.name, "libfakehip.so")


def run(script, timeout=120):
    code = PRELUDE.format(so=build(), root=ROOT, here=HERE) + script
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=timeout, cwd=ROOT)
    assert r.returncode == 0, f"exit {r.returncode}\n{r.stdout[-3000:]}\n{r.stderr[-3000:]}"
    return r.stdout
