"""Host check of the launch arithmetic (csrc/arith.h), compiled by itself: a grid
dimension holds fewer than 2^32 threads, and the workgroups cover their work."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def arith(tmp_path_factory):
    d = tmp_path_factory.mktemp("arith")
    src, lib = str(d / "arith.cpp"), str(d / "arith.so")
    with open(src, "w") as f:
        f.write('#include "arith.h"\n'
                'extern "C" int64_t grid(int64_t n, int64_t per, int t) { return sg::stride_grid(n, per, t); }\n')
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2607_28150_amd", "csrc"), src, "-o", lib], check=True)
    so = ctypes.CDLL(lib)
    so.grid.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    so.grid.restype = ctypes.c_int64
    return so


@pytest.mark.parametrize("per,threads", [(128, 64), (256, 256), (1, 1024)])
def test_stride_grid_fits_a_launch(arith, per, threads):
    for total in (0, 1, per - 1, per, per + 1, 2**31 - 1, 2**31 + 7, 2**33, 2**33 + 1, 2**36, 2**40):
        n = arith.grid(total, per, threads)
        assert 1 <= n and n * threads < 2**32
        # whole cover in one pass wherever a launch may be that large
        assert n * per >= total or (n + 1) * threads >= 2**32
