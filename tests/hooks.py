"""Builds hooks.cpp: host functions of libpwadv that its interface does not
show, callable from tests (no device needed)."""
import ctypes
import os
import subprocess

import pytest

from paper_2301_13016_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


def load(folder):
    """The hooks as a ctypes library built in ``folder``; skips the test where
    libpwadv is not built."""
    try:
        B.lib()
    except B.PWLibraryMissing:
        pytest.skip("library not built")
    out = os.path.join(str(folder), "hooks.so")
    root, pkg = os.path.dirname(HERE), os.path.dirname(B.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-shared", "-fPIC", "-o", out,
                    os.path.join(HERE, "hooks.cpp"), "-I/opt/rocm/include", "-I" + os.path.join(root, "include"),
                    "-I" + os.path.join(pkg, "csrc"), B.LIB_PATH, "-Wl,-rpath," + pkg], check=True)
    return ctypes.CDLL(out)
