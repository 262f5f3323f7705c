"""Which kernel a batched attention launch takes and how it is cut (csrc/la_batch_plan.h, plan_launch: host
code, built here on its own with the host compiler)."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2402_02057_amd import buildlib, workloads as wl

SHIM = r"""
#include <chrono>
#include "la_batch_plan.h"
extern "C" long long launch_end(const int* order, int n, const int* wgs, const long long* cost)
{
    return la::batch_plan::launch_end(order, n, wgs, cost);
}
extern "C" double plan_us(const int* chunks, int n, int tiles, int kv_heads)
{
    double best = 1e9;
    for (int r = 0; r < 20; ++r) {
        const auto from = std::chrono::steady_clock::now();
        volatile int sink = 0;
        for (int k = 0; k < 5; ++k) sink += la::plan_launch(chunks, n, tiles, kv_heads, 128).cuts[0];
        const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - from).count() / 5;
        if (us < best) best = us;
    }
    return best;
}
extern "C" int launch(const int* chunks, int n, int tiles, int kv_heads, int head_dim, int rows, int* cuts, int* place)
{
    const la::LaunchPlan p = la::plan_launch(chunks, n, tiles, kv_heads, head_dim, rows < 0 ? 0 : rows, rows >= 0);
    for (int i = 0; i < n; ++i) { cuts[i] = p.cuts[i]; place[i] = p.place[i]; }
    return p.rows;
}
extern "C" int batch(const int* chunks, int n, int tiles, int kv_heads, int head_dim, int rows, int* cuts, int* place)
{
    const la::BatchPlan p = la::plan_batch(chunks, n, tiles, kv_heads, head_dim, rows);
    for (int i = 0; i < n; ++i) { cuts[i] = p.cuts[i]; place[i] = p.place[i]; }
    return p.rows128 ? 128 : 64;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_plan")
    source, so = d / "shim.cpp", d / "shim.so"
    source.write_text(SHIM)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", buildlib.CSRC,
                    str(source), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.launch_end.restype, lib.plan_us.restype = ctypes.c_longlong, ctypes.c_double
    return lib


def ask(entry, chunks, tiles, kv_heads, head_dim=128, rows=0):
    arr = ctypes.c_int * len(chunks)
    cuts, place = arr(), arr()
    form = entry(arr(*chunks), len(chunks), tiles, kv_heads, head_dim, rows, cuts, place)
    return form, list(cuts), list(place)


def chunks_of(prefixes, T):
    return [-(-P // 64) + -(-T // 64) for P in sorted(prefixes, reverse=True)]


def test_every_plan_can_be_launched(lib):
    """Each step once, no range empty, and partial results of a pipelined launch within what the library
    reserves for one (58 MB; eight waves of 16 KB and 512 bytes each)."""
    rng = random.Random(1)
    taken = 0
    for _ in range(3000):
        T, group, kv_heads = 1 + rng.randint(1, 60) * rng.randint(2, 6), rng.choice([1, 4, 8]), rng.choice([1, 2, 8, 32])
        top = round(64 * 256 ** rng.random())
        chunks = chunks_of([rng.randint(0, top) for _ in range(rng.randint(2, 16))], T)
        tiles, head_dim, rows = -(-T * group // 32), rng.choice([64, 128, 128]), rng.choice([0, 0, 64, 128, 256])
        form, cuts, place = ask(lib.launch, chunks, tiles, kv_heads, head_dim, rows)
        assert sorted(place) == list(range(len(chunks))) and all(1 <= x <= c for x, c in zip(cuts, chunks))
        if form != 256:
            assert (form, cuts, place) == ask(lib.batch, chunks, tiles, kv_heads, head_dim, rows if rows != 256 else 0)
            assert rows != 256 or head_dim == 64 or tiles < 4
            continue
        assert head_dim == 128 and tiles >= 4 and rows in (0, 256)
        taken += rows == 0
        workgroups = sum(kv_heads * -(-tiles // 8) * x for x in cuts if x > 1)
        assert workgroups * 8 * (16384 + 512) <= 58 << 20
    assert taken > 100


@pytest.mark.parametrize("prefixes, T, heads, kv_heads, form, cuts", [
    (wl.ragged_prefix_lengths(), 121, 32, 8, 256, [4, 4, 3, 2, 1, 1, 1, 1]),   # long and ragged: ranges of about equal length
    ([1021 - 37 * i for i in range(16)], 81, 32, 8, 256, [1] * 16),           # a serving batch, uncut
    ([1024] * 8, 121, 32, 32, 128, [1] * 8),                                   # four tiles: nothing to share a chunk with
    ([256] * 4, 121, 32, 8, 64, [1] * 4),
    ([616, 300, 88], 361, 32, 8, 128, [2, 2, 1]),                              # the times too close to call
    ([512] * 6, 41, 32, 8, 64, [1] * 6),                                       # test_gpu_graph.py: an uncut batch, and
    ([512] * 4, 41, 32, 8, 64, [2] * 4),                                       # a smaller one that is cut
    ([8000, 8000], 121, 32, 8, 256, [8, 8]),                                   # test_gpu_workspace.py
], ids=["ragged", "serving", "7b", "small", "wide-windows", "six", "four", "two"])
def test_kernel_and_cuts(lib, prefixes, T, heads, kv_heads, form, cuts):
    got = ask(lib.launch, chunks_of(prefixes, T), -(-T * (heads // kv_heads) // 32), kv_heads)
    assert got[:2] == (form, cuts)


@pytest.mark.parametrize("prefixes, heads, kv_heads, rows, cuts", [
    ([300, 200], 8, 2, 64, [1, 1]), ([4000, 300], 32, 8, 64, [4, 1]), ([300, 200], 4, 1, 128, [1, 1]),
    ([4000, 300], 32, 8, 128, [9, 1]), ([300, 200], 4, 1, 256, [1, 1]), ([4000, 300], 4, 1, 256, [10, 1]),
])
def test_cuts_of_a_forced_form(lib, prefixes, heads, kv_heads, rows, cuts):
    """What test_gpu_row_isolation.py goes by: 81 rows."""
    assert ask(lib.launch, chunks_of(prefixes, 81), -(-81 * (heads // kv_heads) // 32), kv_heads, rows=rows)[:2] == (rows, cuts)


def test_without_the_pipelined_kernel_a_launch_is_the_staged_one(lib):
    """Where its partial results have no room (test_gpu_workspace.py)."""
    for chunks, tiles, kv_heads in drawn(300, seed=13):
        assert ask(lib.launch, chunks, tiles, kv_heads, rows=-1) == ask(lib.batch, chunks, tiles, kv_heads)
    two = chunks_of([8000, 8000], 121)
    assert ask(lib.batch, two, 16, 8)[:2] == (64, [2, 2]) == ask(lib.batch, two, 16, 8, rows=64)[:2]
    assert 16 * 16 * 8 * (16384 + 512) > 32 << 20


def drawn(count, seed):
    rng = random.Random(seed)
    for _ in range(count):
        T, group, kv_heads = 1 + rng.randint(2, 30) * rng.randint(4, 8), rng.choice([1, 4, 8]), rng.choice([1, 2, 8, 10])
        top, n, alike = round(64 * 256 ** rng.random()), rng.randint(2, 16), rng.random() < 0.4
        yield chunks_of([top if alike else rng.randint(0, top) for _ in range(n)], T), -(-T * group // 32), kv_heads


def pipelined_end(lib, chunks, tiles, kv_heads, cuts, place=None):
    """The end of a pipelined launch by the planner's times, and whether it may be launched."""
    blocks = -(-tiles // 8)
    per_block, units, n = -(-tiles // blocks), kv_heads * blocks, len(chunks)
    cost = [-(-c // x) * (72 + 109 * per_block // 8) + 700 + 65 * per_block for c, x in zip(chunks, cuts)]
    order = place or sorted(range(n), key=lambda i: (-cost[i], i))
    wgs, cut = [-(-units * x // 8) for x in cuts], sum(units * x for x in cuts if x > 1)
    end = lib.launch_end((ctypes.c_int * n)(*order), n, (ctypes.c_int * n)(*wgs), (ctypes.c_longlong * n)(*cost))
    return end + (350 + cut if cut else 0), cut <= 448, sum(a * b for a, b in zip(wgs, cost)) // 32 + (350 + cut if cut else 0)


def test_no_pipelined_launch_ends_later_than_if_every_cut_is_placed(lib):
    """The step with the longest ranges is cut once more, down to ranges of seven chunks or until the sum of
    the workgroups alone takes as long as the best launch; the planner passes over most of these sets."""
    for chunks, tiles, kv_heads in drawn(150, seed=11):
        if tiles < 4:
            continue
        cuts, best = [1] * len(chunks), None
        while True:
            end, allowed, least = pipelined_end(lib, chunks, tiles, kv_heads, cuts)
            if not allowed or (best is not None and least >= best):
                break
            best = end if best is None else min(best, end)
            ranges = [-(-c // x) for c, x in zip(chunks, cuts)]
            if max(ranges) < 8:
                break
            cuts[ranges.index(max(ranges))] += 1
        form, cuts, place = ask(lib.launch, chunks, tiles, kv_heads, rows=256)
        end, allowed, _ = pipelined_end(lib, chunks, tiles, kv_heads, cuts, place)
        assert form == 256 and allowed and end <= best, (chunks, tiles, kv_heads, cuts)
        # the kernel chosen without a hook: the pipelined one with these cuts, or the staged one
        free = ask(lib.launch, chunks, tiles, kv_heads)
        assert free == (form, cuts, place) or free == ask(lib.batch, chunks, tiles, kv_heads)


def test_planning_a_launch_takes_less_than_a_launch(lib):
    """It runs in every call, so once per layer.  The quickest of twenty runs; the bounds are three to four times
    what an idle 2.7 GHz core takes."""
    def us(chunks, tiles, kv_heads):
        return lib.plan_us((ctypes.c_int * len(chunks))(*chunks), len(chunks), tiles, kv_heads)
    times = sorted(us(*b) for b in drawn(300, seed=12))
    assert times[len(times) // 2] < 4, times[::30]
    assert times[-1] < 40, times[::30]
    assert us([260] * 16, 8, 1) < 10             # few heads: many cuts
    assert us([65] * 16, 6, 2) < 12
    assert us(chunks_of(wl.ragged_prefix_lengths(), 121), 16, 8) < 6
