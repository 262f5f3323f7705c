"""How a batched attention launch is cut (csrc/la_batch_plan.h, host code): built here on its own with
the host compiler and compared with the rule that bounds it."""
import ctypes
import heapq
import os
import random
import subprocess

import pytest

from paper_2402_02057_amd import buildlib, workloads as wl

SHIM = r"""
#include <chrono>
#include "la_batch_plan.h"
extern "C" int plan(const int* chunks, int n, int tiles, int kv_heads, int head_dim, int rows, int* cuts, int* place)
{
    const la::BatchPlan p = la::plan_batch(chunks, n, tiles, kv_heads, head_dim, rows);
    for (int i = 0; i < n; ++i) { cuts[i] = p.cuts[i]; place[i] = p.place[i]; }
    return p.rows128 ? 128 : 64;
}
extern "C" long long launch_end(const int* order, int n, const int* wgs, const long long* cost)
{
    return la::batch_plan::launch_end(order, n, wgs, cost);
}
extern "C" double plan_us(const int* chunks, int n, int tiles, int kv_heads, int head_dim)
{
    double best = 1e9;
    for (int r = 0; r < 20; ++r) {
        const auto from = std::chrono::steady_clock::now();
        volatile int sink = 0;
        for (int k = 0; k < 5; ++k) sink += la::plan_batch(chunks, n, tiles, kv_heads, head_dim).cuts[0];
        const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - from).count() / 5;
        if (us < best) best = us;
    }
    return best;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_plan")
    source, so = d / "shim.cpp", d / "shim.so"
    source.write_text(SHIM)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", buildlib.CSRC,
                    str(source), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.launch_end.restype, lib.plan_us.restype = ctypes.c_longlong, ctypes.c_double
    return lib


class Batch:
    """Prefixes (longest first) and a step as the launcher hands them to the planner."""

    def __init__(self, prefixes, T, heads, kv_heads, head_dim):
        self.chunks = [-(-P // 64) + -(-T // 64) for P in sorted(prefixes, reverse=True)]
        self.tiles, self.kv_heads, self.head_dim = -(-T * (heads // kv_heads) // 32), kv_heads, head_dim

    def plan(self, lib, rows=0):
        n = len(self.chunks)
        arr = ctypes.c_int * n
        cuts, place = arr(), arr()
        form = lib.plan(arr(*self.chunks), n, self.tiles, self.kv_heads, self.head_dim, rows, cuts, place)
        return form, list(cuts), list(place)

    def units(self, form):
        return self.kv_heads * -(-self.tiles // (form // 32))

    def bound(self):
        """Form and cuts that every plan is at least as accurate as."""
        form = 128 if self.head_dim == 128 and self.tiles >= 3 and len(self.chunks) * self.units(128) >= 192 else 64
        work = sum(self.chunks) * self.units(form)
        target = max(4, -(-work // (256 if len(set(self.chunks)) == 1 else 384)))
        cuts = [max(1, min(-(-c // target), c // 2, 64)) for c in self.chunks]
        return form, [x if self.groups_whole(form, x) else 1 for x in cuts]

    def groups_whole(self, form, cuts):
        """Workgroups are numbered XCD by XCD, the ranges of a row block one after the other: no XCD ends
        inside a group."""
        total = self.units(form) * cuts
        per_xcd = -(-total // 8)
        return all(first // per_xcd == (first + cuts - 1) // per_xcd for first in range(0, total, cuts))


def batches(count, seed, head_dims=(64, 128)):
    rng = random.Random(seed)
    for _ in range(count):
        top, n = round(64 * 256 ** rng.random()), rng.randint(2, 16)
        N, W = rng.choice([3, 4, 5, 7]), rng.choice([1, 3, 5, 10, 15, 30])
        heads, kv_heads = rng.choice([(32, 8), (32, 32), (64, 8), (8, 2), (16, 4), (10, 10), (4, 1)])
        alike = rng.random() < 0.3
        prefixes = [top if alike else rng.randint(0, top) for _ in range(n)]
        yield Batch(prefixes, 1 + 2 * W * (N - 1), heads, kv_heads, rng.choice(head_dims))


def test_no_step_is_less_accurate_than_under_the_bounding_rule(lib):
    """A step that the rule leaves uncut stays uncut (its partial results would be rounded to bf16), and a
    128-row launch stays one (a 64-row workgroup rounds more sums between its key-split waves)."""
    for b in batches(3000, seed=1):
        form, cuts, place = b.plan(lib)
        bound_form, bound = b.bound()
        assert form >= bound_form, (b.chunks, b.tiles, b.kv_heads)
        assert all(1 <= x <= most for x, most in zip(cuts, bound)), (b.chunks, b.tiles, b.kv_heads, cuts, bound)
        assert sorted(place) == list(range(len(cuts)))


def test_head_dim_64_keeps_the_bounding_rule(lib):
    """The times the search goes by are those of the head_dim 128 kernels."""
    for b in batches(500, seed=2, head_dims=(64,)):
        form, cuts, place = b.plan(lib)
        assert (form, cuts) == b.bound(), (b.chunks, b.tiles, b.kv_heads)
        assert place == list(range(len(cuts)))


def test_no_group_lies_on_two_xcds(lib):
    """It would exchange nothing: its last workgroup would compute the rows again over all keys."""
    many = list(batches(2000, seed=3)) + [Batch([4096] * n, T, H, KV, 128) for n in (2, 3, 16) for T in (13, 41, 81)
                                          for H, KV in [(4, 4), (8, 2), (4, 1), (10, 10), (7, 7), (40, 10)]]
    for b in many:
        for rows in (0, 64, 128):
            form, cuts, _ = b.plan(lib, rows)
            assert all(b.groups_whole(form, x) for x in set(cuts)), (b.chunks, b.tiles, b.kv_heads, form, cuts)


@pytest.mark.parametrize("prefixes, W, heads, kv_heads, form, cuts, place", [
    ([256] * 6, 10, 32, 8, 128, [1] * 6, [0, 1, 2, 3, 4, 5]),
    ([256] * 4, 15, 32, 8, 64, [1] * 4, [0, 1, 2, 3]),
    ([2000, 1300, 700, 90, 40], 10, 32, 8, 128, [4, 3, 2, 1, 1], [0, 1, 2, 3, 4]),
    ([1101, 1100, 1099, 130, 64, 0], 5, 8, 2, 64, [1] * 6, [0, 1, 2, 3, 4, 5]),
    ([100] * 16, 5, 64, 64, 64, [1] * 16, list(range(16))),
    ([3000, 900, 800, 700], 5, 32, 8, 64, [5, 2, 2, 1], [0, 3, 1, 2]),
    ([1021 - 37 * i for i in range(16)], 10, 32, 8, 128, [2] * 5 + [1] * 11, [5, 6, 7, 8, 9, 10, 11, 12, 13, 0, 1, 2, 3, 14, 15, 4]),
    ([14559, 13246, 13048, 7849, 2492, 2413, 2180, 1253], 15, 32, 8, 128, [2, 2, 2, 1, 1, 1, 1, 1], [3, 0, 1, 2, 4, 5, 6, 7]),
], ids=["rows128", "rows64", "mixed", "few-heads", "rounds", "reordered", "serving", "ragged"])
def test_form_cuts_and_order(lib, prefixes, W, heads, kv_heads, form, cuts, place):
    assert Batch(prefixes, 1 + 8 * W, heads, kv_heads, 128).plan(lib) == (form, cuts, place)


def ends(lib, b, form, cuts, place):
    fixed, exchange = (6, 1) if form == 128 else (5, 2)
    n, arr = len(cuts), ctypes.c_int * len(cuts)
    wgs = [-(-b.units(form) * x // 8) for x in cuts]
    cost = [-(-c // x) + fixed + (exchange if x > 1 else 0) for c, x in zip(b.chunks, cuts)]
    return lib.launch_end(arr(*place), n, arr(*wgs), (ctypes.c_longlong * n)(*cost)) * (16 if form == 128 else 11)


def test_no_launch_ends_later_than_under_the_bounding_rule(lib):
    """By the planner's own times, with the steps in the order they come, longest prefix first."""
    many = list(batches(2000, seed=8, head_dims=(128,))) + [Batch(wl.ragged_prefix_lengths(), 1 + 8 * W, 32, 8, 128) for W in wl.RAGGED_W]
    for b in many:
        form, cuts = b.bound()
        assert ends(lib, b, *b.plan(lib)) <= ends(lib, b, form, cuts, range(len(cuts))), (b.chunks, b.tiles, b.kv_heads)


def test_longest_ranges_start_first(lib):
    """Cost of a workgroup in chunks: its range, 6 more in the 128-row form and 5 in the 64-row one, and 1
    or 2 for the exchange of a cut step."""
    reordered = 0
    for b in batches(1000, seed=7, head_dims=(128,)):
        form, cuts, place = b.plan(lib)
        cost = [-(-c // x) + (0 if x == 1 else 1 if form == 128 else 2) for c, x in zip(b.chunks, cuts)]
        if place != sorted(place):
            assert all(cost[i] >= cost[j] for i, j in zip(place, place[1:])), (b.chunks, cuts, place)
            reordered += 1
    assert reordered > 50


def test_workspace_of_a_launch_is_bounded(lib):
    """What the library reserves (la_api.hip: 32 MB of partial results, 512 KB of tickets) holds any batch of the staged kernel."""
    for b in batches(2000, seed=6):
        for rows in (0, 64, 128):
            form, cuts, _ = b.plan(lib, rows)
            workgroups = sum(b.units(form) * x for x in cuts if x > 1)
            groups = sum(b.units(form) for x in cuts if x > 1)
            assert workgroups <= 768 and groups <= 384, (b.chunks, b.tiles, b.kv_heads, form, cuts)
    waves, slices = 8, 2                                                        # of a 128-row workgroup, the largest
    assert 768 * waves * (slices * 16 * 64 * 2 + 64 * 8) <= 32 << 20 and 384 * waves * 128 <= 512 << 10


def test_launch_end_is_that_of_placing_workgroups_one_by_one(lib):
    rng = random.Random(4)
    for _ in range(500):
        n = rng.randint(1, 16)
        wgs = [rng.choice([1, 2, 3, 5, 31, 32, 33, 64, rng.randint(1, 200)]) for _ in range(n)]
        cost = [rng.choice([7, 8, 12, rng.randint(1, 300)]) for _ in range(n)]
        order = sorted(range(n), key=lambda i: -cost[i])
        loads = [0] * 32
        for i in order:
            for _ in range(wgs[i]):
                heapq.heapreplace(loads, loads[0] + cost[i])
        got = lib.launch_end((ctypes.c_int * n)(*order), n, (ctypes.c_int * n)(*wgs), (ctypes.c_longlong * n)(*cost))
        assert got == max(loads), (order, wgs, cost)


def test_planning_takes_less_than_a_launch(lib):
    """It runs in every call, so once per layer.  The quickest of twenty runs, and a bound of three times
    what an idle 2.7 GHz core takes for the slowest."""
    def us(b):
        n = len(b.chunks)
        return lib.plan_us((ctypes.c_int * n)(*b.chunks), n, b.tiles, b.kv_heads, b.head_dim)
    times = sorted(us(b) for b in batches(300, seed=5, head_dims=(128,)))
    assert times[len(times) // 2] < 3, times[::30]
    assert times[-1] < 30, times[::30]
    assert us(Batch([4096] * 16, 41, 8, 2, 128)) < 12
