"""Builds and binds tests/device_math.hip (the library's FP64 noise arithmetic over arrays)."""
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1009_0254_amd", "csrc")
LIB = os.path.join(HERE, "libdevice_math.so")
LN, SIN, COS, RCP, DIV, SQRT, ROOT, RROOT = range(8)


def build() -> str:
    from paper_1009_0254_amd import build as B
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *B.FLAGS, "-I", CSRC, os.path.join(HERE, "device_math.hip"), "-o", LIB + ".tmp"],
                   check=True, capture_output=True, text=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


def lib() -> ctypes.CDLL:
    if not os.path.exists(LIB):
        build()
    L = ctypes.CDLL(LIB)
    vp, i = ctypes.c_void_p, ctypes.c_int
    L.device_eval.argtypes = [i, vp, vp, vp, i, vp]
    L.host_eval.argtypes = [i, vp, vp, vp, i]
    L.host_eval.restype = None
    return L
