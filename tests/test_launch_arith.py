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
                'extern "C" int64_t grid(int64_t n, int64_t per, int t) { return sg::stride_grid(n, per, t); }\n'
                'extern "C" int slices(int64_t n, int64_t t, int64_t *out) {\n'
                '    int c = 0;\n'
                '    sg::launch_slices(n, t, [&](int64_t f, int64_t m) { out[2 * c] = f; out[2 * c + 1] = m; ++c; });\n'
                '    return c;\n}\n')
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2607_28150_amd", "csrc"), src, "-o", lib], check=True)
    so = ctypes.CDLL(lib)
    so.grid.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    so.grid.restype = ctypes.c_int64
    so.slices.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    return so


@pytest.mark.parametrize("per,threads", [(128, 64), (256, 256), (1, 1024)])
def test_stride_grid_fits_a_launch(arith, per, threads):
    for total in (0, 1, per - 1, per, per + 1, 2**31 - 1, 2**31 + 7, 2**33, 2**33 + 1, 2**36, 2**40):
        n = arith.grid(total, per, threads)
        assert 1 <= n and n * threads < 2**32
        # whole cover in one pass wherever a launch may be that large
        assert n * per >= total or (n + 1) * threads >= 2**32


@pytest.mark.parametrize("threads", [256, 512, 16 * 512])
def test_launch_slices_cover_their_work(arith, threads):
    most = (2**32 - 1) // threads
    for count in (0, 1, most - 1, most, most + 1, 3 * most + 5):
        out = (ctypes.c_int64 * 16)()
        c = arith.slices(count, threads, out)
        at = 0
        for i in range(c):
            assert out[2 * i] == at and 0 < out[2 * i + 1] and out[2 * i + 1] * threads < 2**32
            at += out[2 * i + 1]
        assert at == count
