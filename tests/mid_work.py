"""The work division of the 64- and 128-row token tiles (csrc/mid_work.h), compiled for the host: what the kernel decides on the
device, by the same text."""
import ctypes
import os
import subprocess
import tempfile

from paper_2503_06823_amd import build as B

HOST = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            out = os.path.join(tmp, "mid_work.so")
            subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", B.CSRC, "-I", os.path.join(B.ROOT, "include"),
                            os.path.join(HOST, "mid_work.cpp"), "-o", out], check=True)
            _lib = ctypes.CDLL(out)
        _lib.cut_share_begin.restype = ctypes.c_uint
    return _lib
