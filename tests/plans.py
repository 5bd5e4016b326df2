"""The kernels' plans on the host: csrc's plan headers compiled with g++ behind
tests/plan_shim.cpp (no GPU, no HIP), so that a test can say which path a call
takes."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_26333_amd", "csrc")
GemvPlan = collections.namedtuple("GemvPlan", "ok BV W CPW KG KCR TPG G park")


@functools.lru_cache(None)
def shim():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan_shim.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC,
                        os.path.join(HERE, "plan_shim.cpp"), "-o", so], check=True)
        lib = ctypes.CDLL(so)   # stays mapped when the file goes
    i64, i32 = ctypes.c_int64, ctypes.c_int
    lib.gemv_contract_groups.argtypes, lib.gemv_contract_groups.restype = [i64] * 4, i64
    lib.gemv_plan.argtypes, lib.gemv_plan.restype = [i32] + [i64] * 5 + [ctypes.POINTER(i64)], None
    lib.gemv_bad_loads.argtypes, lib.gemv_bad_loads.restype = [i32] + [i64] * 6 + [i32], i64
    lib.gemm_short_tile.argtypes, lib.gemm_short_tile.restype = [i64] * 4, i32
    return lib


def gemv_plan(bits, B, N, K, most=None, cus=256):
    """Plan of the batched GEMV kernel; bits 4: NVFP4 weights.  most: K groups
    of the caller's workspace (LUT: the ones of the size query)."""
    T, KC = (N + 15) // 16, (K + 127) // 128
    if most is None:
        most = shim().gemv_contract_groups(B, T, KC, cus)
    out = (ctypes.c_int64 * 9)()
    shim().gemv_plan(bits, B, T, KC, most, cus, out)
    return GemvPlan(*out)


def gemv_bad_loads(bits, B, N, K, most, scales, cus=256):
    return shim().gemv_bad_loads(bits, B, (N + 15) // 16, (K + 127) // 128, (K + 63) // 64, most, cus, scales)


def gemm_short_tile(M, N, K, cus=256):
    """(rows, columns) in 32s of the NVFP4 GEMM's short-grid tile; None: the ring kernels."""
    v = shim().gemm_short_tile(M, N, K, cus)
    return None if v < 0 else divmod(v, 100)
