"""The host arithmetic of the launches (csrc/launch_plan.hpp), compiled on its
own with the host compiler: the cut of the rows into work items, what runs an
iteration's tail, how many iterations are launched in a row, and grids that grow
with the number of packings."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2608_12235_amd._lib import Tuning

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_12235_amd", "csrc")

SOURCE = """
#include "launch_plan.hpp"
using namespace rcp;
extern "C" {
int units_row(const rcp_tuning *t) { return row_units(*t); }
int units_item(const rcp_tuning *t, int waves, int64_t n, int64_t e) { return item_units(*t, waves, n, e); }
int rows_max(const rcp_tuning *t, int waves) { return item_rows_max(*t, waves); }
int64_t slots(const rcp_tuning *t, int waves, int64_t n, int64_t e) { return item_slots(*t, waves, n, e); }
int64_t ahead(int64_t iters, int64_t since_it, int64_t interval, double disp2, double lim,
              int64_t to_limit, int64_t to_end, int64_t K)
{
    return iterations_ahead({iters, since_it, interval, disp2, lim, to_limit, to_end}, K);
}
int64_t left(const int64_t *budget, int n, int rung, int64_t done) { return schedule_left(budget, n, rung, done); }
int64_t per_packing(int64_t nseg, int64_t nmax) { return blocks_per_packing(nseg, nmax); }
int64_t per_scan(int bits) { return packings_per_scan(bits); }
int fused(const rcp_tuning *t, int waves) { return fuses_tail(*t, waves); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), src, "-o", lib], check=True)
    L = C.CDLL(lib)
    L.per_packing.restype = L.per_scan.restype = C.c_int64
    L.per_packing.argtypes = [C.c_int64, C.c_int64]
    L.slots.restype = L.ahead.restype = L.left.restype = C.c_int64
    i64 = C.c_int64
    L.ahead.argtypes = [i64, i64, i64, C.c_double, C.c_double, i64, i64, i64]
    L.left.argtypes = [C.POINTER(i64), C.c_int, C.c_int, i64]
    L.slots.argtypes = L.units_item.argtypes = [C.c_void_p, C.c_int, C.c_int64, C.c_int64]
    return L


def _tuning(**kw):
    t = Tuning()
    t.row_cost, t.item_work, t.variant = 6, 1536, 192
    for k, v in kw.items():
        setattr(t, k, v)
    return t


def _items(plan, t, waves, degrees):
    """Rows of every item of the cut, and the slots there are for them."""
    n, m = len(degrees), int(np.sum(degrees))
    rp = np.concatenate([[0], np.cumsum(degrees)])[:-1]
    w = (plan.units_row(C.byref(t)) * np.arange(n) + rp) // plan.units_item(C.byref(t), waves, n, m)
    return np.bincount(w), plan.slots(C.byref(t), waves, n, m)


@pytest.mark.parametrize("row_cost,item_work,variant", [
    (6, 1536, 192), (6, 3072, 224), (1, 512, 32), (1, 1, 192), (4, 1024, 192), (4, 2048, 32),
    (65536, 65536 * 512, 32), (7, 3583, 32), (64, 16384, 0)])
@pytest.mark.parametrize("n", [1, 64, 2000, 6239, 30011])
def test_items_fit_a_wave_and_the_table(plan, row_cost, item_work, variant, n):
    t = _tuning(row_cost=row_cost, item_work=item_work, variant=variant)
    rng = np.random.default_rng(n)
    for deg in (np.zeros(n, int), np.ones(n, int), rng.integers(0, 3, n), rng.integers(0, 40, n)):
        for waves in (1, 0):
            rows, slots = _items(plan, t, waves, deg)
            assert len(rows) <= slots and slots % 4 == 0
            assert rows.max() <= plan.rows_max(C.byref(t), waves)
            assert rows.max() <= (64 if waves or not variant & 32 else 128)


def test_wide_items_have_more_rows_than_lanes(plan):
    # sparse rows at 6 / 3072: the cut for the 512-row kernel, which a kernel
    # with a row a lane must not be given
    t = _tuning(row_cost=6, item_work=3072, variant=224)
    rows, _ = _items(plan, t, 0, np.zeros(20000, int))
    assert rows.max() == 128 and plan.rows_max(C.byref(t), 0) == 128
    rows, _ = _items(plan, t, 1, np.zeros(20000, int))
    assert rows.max() == 64 and plan.rows_max(C.byref(t), 1) == 64


def test_every_iteration_has_a_tail(plan):
    # a gradient kernel without the fused form must be followed by the tail's
    # own launch: bits 3 and 5 select such kernels, and so do walls, frozen
    # spheres and two dimensions
    for variant in range(256):
        t = _tuning(variant=variant, fused_tail=1)
        assert plan.fused(C.byref(t), 0) == (0 if variant & 8 or variant & 32 else 1), variant
        assert plan.fused(C.byref(t), 1) == 0
        t.fused_tail = 0
        assert plan.fused(C.byref(t), 0) == 0


def test_launches_end_with_the_schedule(plan):
    # a known interval of 400, fresh list: what is left of it, unless a limit
    # or the schedule's end comes first
    far = 1 << 62
    assert plan.ahead(1000, 1000, 400, 0.0, 1.0, far, far, 32) == 400
    assert plan.ahead(1150, 1000, 400, 0.0, 1.0, far, far, 32) == 250
    assert plan.ahead(1150, 1000, 400, 0.0, 1.0, 100, far, 32) == 100
    assert plan.ahead(0, 0, 400, 0.0, 1.0, far, 1, 32) == 1
    assert plan.ahead(0, 0, 0, 0.0, 1.0, far, 5, 32) == 5
    # a build that the schedule's count knows nothing of adds nothing
    assert plan.ahead(0, 900, 400, 0.0, 1.0, far, far, 32) == 400
    # no interval yet: the displacement so far, at most twice as many again
    assert plan.ahead(40, 0, 0, 0.25, 1.0, far, far, 32) == 40
    assert plan.ahead(40, 0, 0, 1e-6, 1.0, far, far, 32) == 80
    assert plan.ahead(40, 0, 0, 4.0, 1.0, far, far, 32) == 0


def test_what_is_left_of_a_schedule(plan):
    b = (C.c_int64 * 4)(10, 20, 1 << 62, 1 << 62)
    assert plan.left(b, 1, 0, 0) == 10 and plan.left(b, 2, 0, 3) == 27 and plan.left(b, 2, 1, 3) == 17
    assert plan.left(b, 1, 0, 25) == 0 and plan.left(b, 0, 0, 0) == 0
    assert plan.left(b, 4, 0, 7) == (1 << 62) - 7 == plan.left(b, 4, 2, 7)


def test_grids_of_many_packings(plan):
    # a launch takes fewer than 2^32 threads along x; 65535 blocks, no more,
    # along y, where a census of 65536 packings would not fit
    for nseg in (1, 2, 16, 8191, 8193, 65535, 65536, 1 << 20):
        for nmax in (1, 256, 257, 100000, 1 << 24):
            per = plan.per_packing(nseg, nmax)
            assert 1 <= per <= max(1, (nmax + 255) // 256)
            assert nseg * per <= max(nseg, 8192) and nseg * per * 256 < 1 << 32
    for bits in range(1, 10):
        assert plan.per_scan(bits) >= 32767
        assert (plan.per_scan(bits) << bits) * 256 < 1 << 32
