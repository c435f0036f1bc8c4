"""Runs a test's body in a child process against the stand-in for the HIP
runtime (hip_stand_in.cpp): no GPU, PyTorch not loaded.  The body sees the
names ``ile``, ``synth``, ``np``, ``fail(name, nth)``, ``clear()`` and
``calls()``, the recorded calls as tuples (name, device, stream's device,
words)."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.modules["torch"] = None
si = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
si.si_log.restype = ctypes.c_char_p
sys.path.insert(0, {root!r})
import numpy as np
from paper_1902_04934_amd import ile, synth


def fail(name, nth=1):
    si.si_fail(name.encode(), nth)


def clear():
    si.si_clear()


def calls():
    out = []
    for line in si.si_log().decode().splitlines():
        name, dev, sdev, *words = line.split()
        out.append((name, int(dev), int(sdev), words))
    return out


def names(kinds=None):
    return [c[0] if c[0] != "hipLaunchKernel" else c[3][0] for c in calls()
            if kinds is None or c[0] in kinds]


"""


def run(tmp_path, body):
    if not (shutil.which("g++") and os.path.exists("/opt/rocm/include/hip/hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not installed")
    lib = str(tmp_path / "libhip_stand_in.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "hip_stand_in.cpp"), "-o", lib],
                   check=True)
    if "ILE_LIB" not in os.environ:
        from paper_1902_04934_amd import build
        if not os.path.exists(build.LIB):
            build.build()
    code = PRELUDE.format(lib=lib, root=ROOT) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout
