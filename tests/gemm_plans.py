"""The plans of a bf16 model's projections (csrc/gemm_plan.cpp built with g++),
so that a GPU test can state, and assert, which kernels its sizes reach."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_12243_amd", "csrc")
ROLES = ("qkv", "o", "gate_up", "down", "head")
PATHS = ("stream", "row_tile", "prefill", "head", "f32")


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plans.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host", "gemm_plan_shim.cpp"), os.path.join(CSRC, "gemm_plan.cpp"),
                        "-o", so], check=True)
        return C.CDLL(so)


def _shape(m, role):
    d, hd = m["d_model"], m["head_dim"]
    return {"qkv": ((m["n_heads"] + 2 * m["n_kv_heads"]) * hd, d), "o": (d, m["n_heads"] * hd),
            "gate_up": (2 * m["d_ffn"], d), "down": (d, m["d_ffn"]), "head": (m["vocab"], d)}[role]


def path(m, role, M):
    """Kernel family of a projection of a forward of M rows (head: M head rows)."""
    return PATHS[_lib().plan_path(ROLES.index(role), M, *_shape(m, role))]


def tile(m, role, M):
    """(rows, columns, K splits) of the row-tile kernel."""
    r, c, k = C.c_int(), C.c_int(), C.c_int()
    _lib().plan_tile(ROLES.index(role), M, *_shape(m, role), C.byref(r), C.byref(c), C.byref(k))
    return r.value, c.value, k.value
