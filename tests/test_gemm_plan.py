"""CPU tests of the projections' plans: kernel family, tile and K splits by row
count, and the workspace that holds the split-K partial products.

The C++ test (tests/host/gemm_plan_test.cpp, built with g++ under
UndefinedBehaviorSanitizer) goes over every row count of
several model shapes; via_workspace_bytes is checked through the library.
"""
import ctypes as C
import os
import shutil
import subprocess

import pytest

from paper_2606_12243_amd import via
from workload import configs

import row_tile_cases

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_12243_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_gemm_plan_under_sanitizer(tmp_path):
    exe = tmp_path / "gemm_plan_test"
    cmd = ["g++", "-std=c++17", "-O2", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "gemm_plan_test.cpp"), os.path.join(CSRC, "gemm_plan.cpp"),
           "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("name", ["8b_bf16_chain", "1b_bf16"])
def test_workspace_grows_with_max_rows(name):
    """A handle for more rows needs no less workspace (every region is at least
    as large, so a forward of fewer rows fits wherever a smaller handle held it)."""
    d = via.model_desc(configs.get(name)["model"])
    sizes = [via.via_workspace_bytes(C.byref(d), r, 4, 8, 8, 4) for r in range(1, 700)]
    assert sizes[0] > 0
    assert [r + 1 for r in range(1, len(sizes)) if sizes[r] < sizes[r - 1]] == []


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_gpu_cases_reach_every_row_tile_form():
    """The sizes that the GPU tests run take every (tile, K groups, epilogue) the library holds."""
    taken = set().union(*(row_tile_cases.forms(n, r) for n, r in row_tile_cases.CASES))
    assert taken == row_tile_cases.ALL_FORMS
