"""The work division of the 64- and 128-row token tiles (csrc/mid_work.h), compiled for the host: what the kernel decides on the
device, by the same text."""
import ctypes
import os
import subprocess
import tempfile
from typing import NamedTuple

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


class Tiles(NamedTuple):
    fewest: int          # column tiles as wide as a tile can hold
    widest: int
    n: int               # the chosen ones
    columns: int
    cut: bool            # along K
    rows: int            # token rows and weight rows of a tile
    weight_rows: int
    persist: bool
    m_tiles: int


def product_tiles(swiglu, counts, N, K, cus=256, ulps=0) -> Tiles:
    """The tiles of a product of N columns and K inputs over slots of `counts` rows."""
    out = (ctypes.c_int * 9)()
    lib().product_tiles(ctypes.c_bool(swiglu), (ctypes.c_int * len(counts))(*map(int, counts)), len(counts), N, K, cus, ulps, out)
    v = list(out)
    return Tiles(*v[:4], bool(v[4]), v[5], v[6], bool(v[7]), v[8])
