"""Builds and loads ``libgolden_open.so`` (golden_open.hip)."""
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SO = os.path.join(HERE, "libgolden_open.so")


def build() -> None:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-fPIC", "-shared", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    os.path.join(HERE, "golden_open.hip"), "-o", SO + ".tmp"], check=True, capture_output=True)
    os.replace(SO + ".tmp", SO)


def lib() -> ctypes.CDLL:
    if not os.path.exists(SO):
        build()
    so = ctypes.CDLL(SO)
    so.golden_scan_and_rows.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                        ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    so.golden_open_mark.restype = ctypes.c_uint32
    return so
