"""Builds host_plans.cpp (the kernels' launch planning as host functions, from the library's
headers and the built library) and loads it."""

import ctypes as C
import os
import subprocess

from paper_2609_30846_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def load(work_dir):
    """The host functions, compiled into ``work_dir`` (no device code, no GPU needed)."""
    out = os.path.join(work_dir, "host_plans.so")
    subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++20", "-fPIC", "-shared", "-I", B.CSRC,
                    "-I", os.path.join(B.ROOT, "include"), os.path.join(HERE, "host_plans.cpp"), "-x", "none", B.LIB,
                    "-Wl,-rpath," + B.HERE, "-o", out],
                   check=True, capture_output=True, text=True)
    lib = C.CDLL(out)
    lib.tile_grid_fault.argtypes = [C.c_int] * 5
    lib.tile_grid_fault.restype = C.c_int64
    lib.div_fault.argtypes = [C.c_uint32, C.c_void_p, C.c_int64]
    lib.div_fault.restype = C.c_int64
    lib.gemm_shape.argtypes = [C.c_void_p] + [C.c_int] * 4 + [C.POINTER(C.c_int)] * 2
    lib.gemm_shape.restype = None
    lib.attn_shape.argtypes = [C.c_int, C.c_int, C.c_int64, C.c_void_p]
    lib.attn_shape.restype = None
    return lib


PLAIN, RESID, SWISH = range(3)  # Epilogue of gemm_tiles.h


def gemm_shape(lib, products, K, epilogue, min_tm=32):
    """(channels, tokens) of the tiles of one launch of ``products`` [(nb, rows, N), ...]."""
    flat = [v for p in products for v in p]
    tn, tm = C.c_int(), C.c_int()
    lib.gemm_shape((C.c_int * len(flat))(*flat), len(products), K, min_tm, epilogue, C.byref(tn), C.byref(tm))
    return tn.value, tm.value


def attn_shape(lib, B, T, d, H):
    """(first shape, second shape or None, paired) of the attention core for a block call, a
    shape being (key splits, 16-query tiles per wave); (None, None, False): spilling workgroups."""
    v = (C.c_int * 7)()
    lib.attn_shape(d // H, T, B * H, v)
    return ((v[0], v[1]) if v[0] else None), ((v[3], v[4]) if v[3] else None), bool(v[6])
