"""Steps alone whose keys are cut into ranges, with any number of row blocks: the ranges of a row block on one XCD (the
mapping of csrc/la_batch_plan.h, on the CPU), and on the GPU no group computed again and none further off."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import la_oracle as orc
from paper_2402_02057_amd import binding, buildlib, workloads as wl

TOL = 2e-2
SHIM = """
#include "la_batch_plan.h"
extern "C" int per_xcd(int units) { return la::step_units_per_xcd(units); }
extern "C" int cuts(int units, int chunks) { return la::step_cuts(units, chunks); }
extern "C" int even(int units, int chunks) { return la::step_cuts_even(units, chunks); }
extern "C" int rows128(int chunks, int tiles, int kv_heads) { return la::step_rows128(chunks, tiles, kv_heads, true, false); }
extern "C" int ranges(int units, int chunks, int rows, int head_dim, int fp32)
{
    const la::StepRanges r = la::step_ranges(units, chunks, rows, head_dim, fp32);
    return r.fp32 ? -r.x : r.x;
}
"""


def test_the_ranges_of_a_row_block_are_on_one_xcd(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", buildlib.CSRC,
                    str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so")], check=True)
    lib = ctypes.CDLL(str(tmp_path / "shim.so"))
    for units in list(range(1, 130)) + [255, 256, 257, 1000]:
        for chunks in (1, 2, 3, 7, 30, 129, 1000):
            x, most = lib.cuts(units, chunks), lib.per_xcd(units)
            if lib.even(units, chunks):
                assert x == 256 // units or x == chunks // 2 or x == 64      # as many ranges as fill the compute units
            assert 1 <= x <= max(1, chunks // 2) and x <= 64 and most * 8 >= units
            for rows, d in ((32, 128), (64, 128), (128, 128), (32, 64), (64, 64)):
                for fp32 in (0, 1):                     # fewer only in fp32, which stays so
                    n = lib.ranges(units, chunks, rows, d, fp32)
                    assert n == x if n > 0 else 2 <= -n <= x and (fp32 or -n < x)
                    assert n < 0 or not fp32 or x == 1
            if x == 1:
                continue
            assert most * x <= 32                       # one round: the compute units of an XCD
            seen = [[] for _ in range(8)]
            for group in range(8 * most * x):           # the kernel's mapping: id -> XCD and slot -> row block and range
                logical = (group & 7) * most * x + (group >> 3)
                if logical < units * x:
                    seen[group & 7].append(logical)
            assert sorted(sum(seen, [])) == list(range(units * x))
            for of_xcd in seen:
                assert len(of_xcd) % x == 0 and all(l // x == of_xcd[i - i % x] // x for i, l in enumerate(of_xcd))
    assert not lib.rows128(66, 31, 1) and not lib.rows128(258, 31, 2)       # few KV heads: 64 rows again
    assert lib.rows128(66, 31, 4) and lib.rows128(514, 31, 2)              # cut 8 times; to 33 chunks
    assert lib.ranges(8, 66, 64, 128, 0) == -11 and lib.ranges(8, 18, 64, 128, 0) == 9 and lib.ranges(8, 258, 64, 128, 0) == 32


SHAPES = [(700, 5, 4, 5, 4, 4, 128),       # 4 row blocks of 32 rows, 5 ranges each
          (2500, 20, 5, 20, 4, 4, 128),    # 12 of 64 rows, 16
          (3000, 10, 5, 10, 10, 10, 128),  # 20, 10
          (900, 5, 4, 5, 4, 4, 64),
          (2500, 20, 5, 20, 4, 4, 64),
          (300, 15, 5, 15, 50, 50, 128)]   # 100, 2
FEWER = [(4096, 15, 5, 15, 4, 4, 128),     # 8 row blocks: 11 ranges in fp32, 32 in bf16 before
         (3900, 3, 4, 1, 32, 8, 128),
         (4096, 15, 5, 15, 4, 4, 64),
         (4096, 15, 5, 15, 8, 1, 128),     # 16 of 64 rows, 8 of 128 before
         (4096, 16, 5, 15, 16, 2, 128)]


def new_like(q):
    return torch.full_like(q, float("nan"))


def error(out, want):
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "P%d-W%d-%d/%d-d%d" % (s[0], s[1], s[4], s[5], s[6]))
def test_every_entry_point_agrees_and_none_is_further_off(shape, override):
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    T, rng = 1 + (W + G) * (N - 1), np.random.default_rng(P)
    x = {k: wl.f32_to_bf16_bits(rng.standard_normal(size=s, dtype=np.float32))
         for k, s in dict(q=(T, H, d), k_cache=(KV, P, d), v_cache=(KV, P, d), step_k=(T, KV, d), step_v=(T, KV, d)).items()}
    dev = {k: binding.bf16_tensor(v) for k, v in x.items()}
    q, cache, args = dev["q"], (dev["k_cache"], dev["v_cache"]), (dev["step_k"], dev["step_v"], P, W, N, G, H, KV, d)
    override("attn_rowtile", "0")
    out = binding.la_step_attention(q, *cache, *args, new_like(q))
    want = orc.step_attention(x["q"], x["k_cache"], x["v_cache"], x["step_k"], x["step_v"], P, W, N, G, H, KV, d)
    err = error(out, want)
    # the same bits again, without an allocation, with room behind the prefix, from pages, as rows, and turned by nothing
    assert torch.equal(out, binding.la_step_attention(q, *cache, *args, new_like(q)))
    assert torch.equal(out, binding.la_step_attention_noalloc(q, *cache, *args, new_like(q)))
    room = [torch.cat([t, torch.full((KV, 70, d), float("nan"), dtype=torch.bfloat16, device="cuda")], 1) for t in cache]
    assert torch.equal(out, binding.la_step_attention_cap(q, *room, *args, new_like(q)))
    n = -(-P // 64)
    table = torch.randperm(n + 3, device="cuda")[:n]
    pages = []
    for t in cache:
        padded = torch.full((KV, n * 64, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        padded[:, :P] = t
        pages.append(torch.full((n + 3, KV, 64, d), float("nan"), dtype=torch.bfloat16, device="cuda"))
        pages[-1][table] = padded.view(KV, n, 64, d).transpose(0, 1)
    assert torch.equal(out, binding.la_step_attention_paged(q, *pages, table.int(), *args, new_like(q)))
    ids = torch.arange(T, dtype=torch.int32, device="cuda")
    assert torch.equal(out, binding.la_step_attention_rows(q, *cache, dev["step_k"], dev["step_v"], ids, *args[2:], new_like(q)))
    cos = torch.ones(P + W + N, d // 2, device="cuda")
    assert torch.equal(out, binding.la_step_attention_rope(q, *cache, dev["step_k"], dev["step_v"], cos, torch.zeros_like(cos), *args[2:], new_like(q)))
    # groups spread over XCDs are computed again, over all keys and without partial results: that is no nearer
    override("force_recompute", "1")
    assert err <= error(binding.la_step_attention(q, *cache, *args, new_like(q)), want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FEWER, ids=lambda s: "P%d-W%d-%d/%d-d%d" % (s[0], s[1], s[4], s[5], s[6]))
def test_fewer_ranges_are_no_further_off_than_all(shape, override):
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    T, rng = 1 + (W + G) * (N - 1), np.random.default_rng(P)
    x = [wl.f32_to_bf16_bits(rng.standard_normal(size=s, dtype=np.float32)) for s in ((T, H, d), (KV, P, d), (KV, P, d), (T, KV, d), (T, KV, d))]
    dev = [binding.bf16_tensor(v) for v in x]
    want = orc.step_attention(*x, P, W, N, G, H, KV, d)
    out = binding.la_step_attention(*dev, P, W, N, G, H, KV, d, new_like(dev[0]))
    assert torch.equal(out, binding.la_step_attention_noalloc(*dev, P, W, N, G, H, KV, d, new_like(dev[0])))
    override("attn_plan", "4,2,0,4,64" if T * H // KV > 480 else "2,4,0,4,64" if d == 128 else "2,2,0,4,64")
    assert error(out, want) <= error(binding.la_step_attention(*dev, P, W, N, G, H, KV, d, new_like(dev[0])), want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES[:5:2], ids=lambda s: "P%d-W%d-%d/%d-d%d" % (s[0], s[1], s[4], s[5], s[6]))
def test_quantised_cache(shape, override):
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    T, gen = 1 + (W + G) * (N - 1), torch.Generator(device="cuda").manual_seed(P)

    def codes(*s):
        return torch.randn(s, device="cuda", generator=gen).mul_(112).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    q = torch.randn(T, H, d, device="cuda", generator=gen).bfloat16()
    kc, vc, sk, sv = codes(KV, P, d), codes(KV, P, d), codes(T, KV, d), codes(T, KV, d)
    scale = torch.full((2, KV), 4 / 448, device="cuda") * (0.75 + 0.5 * torch.rand(2, KV, device="cuda", generator=gen))
    want = orc.step_attention_fp8kv(binding.bf16_bits(q), *(t.cpu().numpy() for t in (kc, vc, sk, sv)), scale[0].cpu().numpy(),
                                    scale[1].cpu().numpy(), P, W, N, G, H, KV, d)
    errors = []
    for again in (None, "1"):
        override("force_recompute", again)
        errors.append(error(binding.la_step_attention_fp8kv(q, kc, vc, sk, sv, scale[0], scale[1], P, W, N, G, H, KV, d, new_like(q)), want))
    assert errors[0] <= errors[1]
