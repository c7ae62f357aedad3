"""Builds and loads the test library of native/radix_wide.hip (for gfx950)."""

import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "radix_wide.hip")
LIB = os.path.join(HERE, "native", "libradix_wide.so")


def build() -> str:
    from paper_2609_21848_amd.build import FLAGS, hipcc
    tmp = f"{LIB}.tmp{os.getpid()}"
    subprocess.run([hipcc(), *FLAGS, "-shared", "-o", tmp, SRC], check=True, capture_output=True)
    os.replace(tmp, LIB)
    return LIB


def load() -> ctypes.CDLL:
    lib = ctypes.CDLL(LIB if os.path.exists(LIB) else build())
    vp = ctypes.c_void_p
    lib.radix_wide_sort.argtypes = [vp, ctypes.c_int64, ctypes.c_int, vp, vp]
    return lib
