"""The encode's emission plan (host code), over every dictionary size and k."""
import ctypes
import math
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_22595_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "emit_plan.hpp"\n'
                   'extern "C" void plan(int m, int k, int w, int* cap, int* lo, float* z) {\n'
                   '    const xmix::EmitPlan e = xmix::emit_plan(m, k, w);\n'
                   '    *cap = e.cap; *lo = e.lo; *z = e.z;\n}\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(lib)], check=True)
    f = ctypes.CDLL(str(lib)).plan

    def call(m, k, w):
        cap, lo, z = ctypes.c_int(), ctypes.c_int(), ctypes.c_float()
        f(m, k, w, ctypes.byref(cap), ctypes.byref(lo), ctypes.byref(z))
        return cap.value, lo.value, z.value
    return call


def sizes(most):
    ms = [*range(256, 8193, 256), 9984, 16384, 16640, 32768, 65536, 131072]
    return [(m, k) for m in ms if m <= most
            for k in (1, 2, 3, 4, 6, 8, 9, 10, 12, 16, 24, 32, 48, 63, 64) if (m // 256) * k <= 16384]


@pytest.mark.parametrize("width,most", [(256, 131072), (128, 32768), (64, 16384)])
def test_window_of_every_plan(plan, width, most):
    """A count the threshold search can settle on: a window of at least two thirds
    of the capacity (two thirds for the tiles that must supply k between them),
    the k values supplied by the bound or expected with room to spare, and a first
    guess inside the window."""
    for m, k in sizes(most):
        cap, lo, z = plan(m, k, width)
        n = m // width
        guess = 0.5 * math.erfc(z / math.sqrt(2)) * width
        assert 0 <= lo <= k and 8 <= cap <= 64 and cap % 4 == 0
        assert 1.99 < guess < cap and guess > lo or n * cap == k, (m, k)
        if lo:
            assert lo * n >= k or lo == k
            if n > 2:
                assert cap - lo >= 2 * cap / 3 - 1, (m, k, lo, cap)
        else:
            assert n * guess - k >= 3.99 * math.sqrt(n * guess), (m, k)


def test_no_bound_where_two_a_tile_are_four_times_k(plan):
    """From 4096 latents on, whole tiles have no lower bound where two values of
    each are four times k: such a bound made every tile search."""
    for m, k in sizes(131072):
        if m >= 4096 and 2 * (m // 256) >= 4 * k:
            assert plan(m, k, 256)[1] == 0, (m, k)
