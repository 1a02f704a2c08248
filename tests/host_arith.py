"""The library's per-particle arithmetic compiled for the host: it is written
for both (GCB_HD), so that its values can be checked without a GPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_14401_amd", "csrc")


def compile_host(tmp, source: str, *flags) -> ctypes.CDLL:
    """A shared library of `source` (host code that includes the headers)."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, lib = os.path.join(tmp, "host.hip"), os.path.join(tmp, "host.so")
    with open(src, "w") as f:
        f.write(source)
    cmd = [hipcc, "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-mfma",
           "-I", CSRC, *flags, src, "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ctypes.CDLL(lib)
