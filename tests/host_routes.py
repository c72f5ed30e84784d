"""Builds a small C++ probe against the library's host code (fwi_host.cpp,
fwi_batch.cpp) and the host-only HIP stand-in of tests/host_asan, to look at the
decisions that the host code makes.  TEST INFRASTRUCTURE ONLY."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_20513_amd", "csrc")
ASAN = os.path.join(ROOT, "tests", "host_asan")


def build(tmp, name, code, defines=()):
    """A shared library of the host code, the stand-in (compiled with `defines`, so that
    `code` can take the place of some of its functions) and `code`."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, stub, so = tmp / (name + ".cpp"), tmp / (name + "_stub.o"), tmp / (name + ".so")
    src.write_text(code)
    flags = ["-std=c++17", "-O1", "-fPIC", "-pthread", "-Wall", "-Wno-unused-function", "-I", ASAN,
             "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    subprocess.run([cxx, *flags, *["-D" + d for d in defines], "-c",
                    os.path.join(ASAN, "hip_host_stub.cpp"), "-o", str(stub)], check=True)
    subprocess.run([cxx, *flags, "-shared", str(src), str(stub), os.path.join(CSRC, "fwi_host.cpp"),
                    os.path.join(CSRC, "fwi_batch.cpp"), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))
