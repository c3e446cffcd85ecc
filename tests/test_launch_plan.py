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
void w_near_joint(int64_t *cur, const int64_t *need) {
    const NearLayout j = near_joint(NearLayout{cur[0], cur[1], cur[2]}, NearLayout{need[0], need[1], need[2]});
    cur[0] = j.tcap, cur[1] = j.vstride, cur[2] = j.hstride;
}
int w_near_fills(int64_t n, int64_t nv, int64_t nh, int64_t roots, int64_t stack, int64_t resident, double budget) {
    return near_fills_device(NearNeed{{n, nv, nh}, roots, stack, 1}, resident, budget);
}
int w_near_stack_records(double nf, double share, int cap, int all) { return near_stack_records(nf, share, cap, all); }
int64_t w_near_waves(int64_t tcap, int64_t vstride, int64_t hstride, int64_t roots, int64_t stack, int64_t waves,
                     double budget, double free_bytes, const double *held) {
    return near_waves(NearNeed{{tcap, vstride, hstride}, roots, stack, waves}, budget, free_bytes, held);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "wrap.cpp", d / "libplan.so"
    src.write_text(WRAP)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2404_19751_amd", "csrc"), str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    I, D = ctypes.c_int64, ctypes.c_double
    L.w_near_stack_records.argtypes = [D, D, ctypes.c_int, ctypes.c_int]
    L.w_near_fills.argtypes = [I] * 6 + [D]
    L.w_near_waves.argtypes = [I] * 6 + [D, D, ctypes.POINTER(D)]
    L.w_near_waves.restype = I
    return L


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


def near(plan, tcap, vstride, hstride, roots, stack, waves, budget=40e9, free=1e18, held=(0,) * 6):
    return plan.w_near_waves(tcap, vstride, hstride, roots, stack, waves, budget, free, (ctypes.c_double * 6)(*held))


def wave_bytes(tcap, vstride, hstride, roots, stack):
    area = ((32 * tcap + 4 * tcap + 15) // 16 * 16 + 8 * 4096 + 255) // 256 * 256
    return [stack, roots, area, 8 * vstride, 8 * hstride, 4]


@pytest.mark.parametrize("tcap", [1, 100, 8192, 466000, 4000000])
@pytest.mark.parametrize("free", [1e6, 3e8, 3e9, 3e10, 1e18])
def test_near_waves_fit(plan, tcap, free):
    """As many wavefronts as run, budget and free memory allow, at least one,
    and one more would not fit."""
    lay = (tcap, 2324, 13944, 90112, 64 * 16384)
    b = wave_bytes(*lay)
    held = [1e8, 0, 2e8, 0, 0, 0]
    n = near(plan, *lay, 2048, free=free, held=held)
    assert 1 <= n <= 2048

    def growth(k):
        return sum(max(0.0, 1.25 * k * x - h) for x, h in zip(b, held) if k * x > h)
    assert n == 1 or (n * sum(b) <= 40e9 and growth(n) <= 0.9 * free)
    assert n == 2048 or (n + 1) * sum(b) > 40e9 or growth(n + 1) > 0.9 * free


def test_near_waves_held_memory_counts(plan):
    lay = (8192, 2324, 13944, 90112, 64 * 16384)
    held = [2048 * x for x in wave_bytes(*lay)]
    assert near(plan, *lay, 2048, free=0.0, held=held) == 2048  # nothing has to grow


def test_near_stack_records(plan):
    f = plan.w_near_stack_records
    assert f(4648, 0.007, 16384, 262144) == 16384  # a narrow cutoff: the depth-first depth
    assert f(4648, 0.007, 64, 262144) == 1024
    for nf in (320, 20480, 81920, 10 ** 6):
        for share in (0.01, 0.3, 0.55, 1.0, 7.0):
            n = f(nf, share, 16384, 262144)
            assert 16384 <= n <= 262144 and (n >= 8 * nf * min(1.0, share) or n == 262144)
    assert f(10 ** 6, 0.9, 1 << 20, 262144) == 1 << 20  # a caller's larger depth stands


def test_layouts_used_in_turn_settle(plan):
    """Surfaces and particle counts in turn prepare tables a few times, then no
    more; a layout always holds what the pass needs."""
    I3 = ctypes.c_int64 * 3
    needs = [(8192, 2324, 13944), (1000, 10242, 0), (8200, 2324, 13944), (500, 642, 3840)]
    cur, changes = I3(0, 0, 0), 0
    for k in range(40):
        need, was = needs[k % 4], list(cur)
        plan.w_near_joint(cur, I3(*need))
        assert all(c >= n for c, n in zip(cur, need))
        changes += list(cur) != was
    assert changes <= 4
    # particles added one at a time: the tables grow by quarters
    cur, changes = I3(1000, 642, 0), 0
    for n in range(1000, 10000):
        was = cur[0]
        plan.w_near_joint(cur, I3(n, 642, 0))
        assert cur[0] >= n
        changes += cur[0] != was
    assert changes <= 12


def test_large_surfaces_stay_on_the_cutoff_kernel(plan):
    """Sphere of 81,920 faces, 16,384 records a stack: half of 2048 wavefronts
    fit the budget up to about a million particles."""
    def fills(n, resident=2048):
        return bool(plan.w_near_fills(n, 40962, 0, 256, 64 * 16384, resident, 40e9))
    assert fills(100) and fills(8192) and fills(466000) and fills(900000)
    assert not fills(1200000) and not fills(4000000)
    assert fills(1200000, 256)
