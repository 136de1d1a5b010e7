"""Host check of the launch and sampling arithmetic (csrc/arith.h), compiled by
itself: a grid dimension holds fewer than 2^32 threads, the workgroups cover
their work, and the sampled keys are spread over all keys and phases."""
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
                '    return c;\n}\n'
                'extern "C" int key(int i, int ns, int seen) { return sg::sample_key(i, ns, seen); }\n')
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


@pytest.mark.parametrize("ns", [512, 640, 1024, 2048])
@pytest.mark.parametrize("ratio", [1, 1.002, 1.5, 1.998, 3.99, 16, 37.3, 4000, 2**18])
def test_sample_keys_are_spread(arith, ns, ratio):
    seen = int(ns * ratio)
    keys = [arith.key(i, ns, seen) for i in range(ns)]
    assert keys == sorted(keys) and keys[0] >= 0 and keys[-1] < seen
    if seen == ns:
        assert keys == list(range(ns))
    # one key in each of ns equal stretches (a rounding of the stretch's ends
    # aside), so every stretch of the prompt has its share, the last keys too
    slack = 1 + seen * 2.0**-22
    assert all(i * seen / ns - slack <= x <= (i + 1) * seen / ns + slack for i, x in enumerate(keys))


@pytest.mark.parametrize("ns,seen", [(512, 8129), (512, 8192), (1024, 16384), (2048, 32705)])
@pytest.mark.parametrize("period", [2, 3, 8, 16, 32, 64])
def test_sample_keys_take_every_phase(arith, ns, seen, period):
    """Keys whose logits repeat are sampled at every phase alike: each phase's
    count within five standard deviations of its share."""
    n = [0] * period
    for i in range(ns):
        n[arith.key(i, ns, seen) % period] += 1
    share = ns / period
    assert max(abs(x - share) for x in n) <= 5 * share**0.5, n
