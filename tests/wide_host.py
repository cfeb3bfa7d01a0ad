"""Builds and loads tests/wide_host.cpp: the host side of csrc/wide.h."""
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


def load(directory) -> ctypes.CDLL:
    so = os.path.join(str(directory), "wide_host.so")
    subprocess.check_call([CLANG, "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           os.path.join(HERE, "wide_host.cpp"), "-o", so])
    return ctypes.CDLL(so)
