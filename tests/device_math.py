"""Builds and loads ``libdevmath.so``: the device arithmetic of ``device_math_check.hip`` behind a C ABI."""
import ctypes
import os
import subprocess

from paper_2402_10914_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "libdevmath.so")


def build() -> str:
    tmp = OUT + ".tmp"
    subprocess.run([hipbuild.HIPCC] + hipbuild.FLAGS + [os.path.join(HERE, "device_math_check.hip"), "-o", tmp], check=True)
    os.replace(tmp, OUT)
    return OUT


def load():
    if not os.path.exists(OUT):
        build()
    L = ctypes.CDLL(OUT)
    for name, n in (("dm_f64", 4), ("dm_f32", 3), ("dm_all_f32", 1)):
        f = getattr(L, name)
        f.restype = ctypes.c_int
        f.argtypes = [ctypes.c_void_p] * n + ([ctypes.c_int] if n > 1 else [])
    L.dm_quotient.restype = ctypes.c_int
    L.dm_quotient.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_double, ctypes.c_int]
    return L
