"""Host arithmetic of launches and scratch memory, compiled from its header
with the host compiler and checked at sizes that no device run allocates."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WRAP = """
#include "launch_plan.h"
using namespace gsim;
extern "C" {
int w_fill_blocks(int64_t n, int block) { return fill_blocks(n, block); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "wrap.cpp", d / "libplan.so"
    src.write_text(WRAP)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2404_19751_amd", "csrc"), str(src), "-o", str(so)])
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("n", [1, 255, 256, 257, 10 ** 6, 2 ** 28, 2 ** 28 + 1, 2048 * (36 * 466000 + 32768) // 8,
                               2 ** 32, 5 * 10 ** 9])
def test_fills_stay_within_a_launch(plan, n):
    """The near tables of 466,000 particles are 4.3e9 words, more than the
    threads of one launch."""
    plan.w_fill_blocks.argtypes = [ctypes.c_int64, ctypes.c_int]
    b = plan.w_fill_blocks(n, 256)
    assert 1 <= b and b * 256 < 2 ** 32
    # every item is reached: one per thread, or by strides of the whole grid
    assert b * 256 >= n or b == 2 ** 20
