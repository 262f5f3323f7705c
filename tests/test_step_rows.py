"""Steps alone that take 128-row workgroups: where the rule draws the line (csrc/la_batch_plan.h, on the CPU), and
on the GPU the steps on its other side, cut with fp32 partial results, cut with bf16 ones and whole."""
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
extern "C" int rows128(int chunks, int tiles, int kv_heads, int many, int codes) { return la::step_rows128(chunks, tiles, kv_heads, many, codes); }
extern "C" int cuts(int units, int chunks) { return la::step_cuts(units, chunks); }
extern "C" int most(int groups) { return groups ? la::kMaxStepGroups : la::kMaxStepWorkgroups; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("step_rows")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", buildlib.CSRC,
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


def ask(lib, P, W, N, G, H, KV, codes=0):
    T = 1 + (W + G) * (N - 1)
    tiles, many = (T * H // KV + 31) // 32, T * H // KV > 480 and (P + T) // 64 >= 64
    return lib.rows128(-(-P // 64) + -(-T // 64), tiles, KV, int(many), codes)


def test_the_rule(lib):
    for s in (wl.LLAMA2_7B, wl.LLAMA2_7B_P256, wl.LLAMA2_13B, wl.LLAMA2_70B):     # latency-bound: 64 rows
        assert not ask(lib, s.P, s.W, s.N, s.G, s.heads, s.kv_heads)
    assert ask(lib, 14559, 15, 5, 15, 32, 8)                    # many rows on a long prefix: as ever
    assert ask(lib, 3719, 17, 5, 16, 32, 32)                    # 96 units fill 192 compute units, 64 fill 256
    assert ask(lib, 60, 30, 7, 30, 64, 8)                       # 368 workgroups in two rounds, 184 in one
    assert ask(lib, 2100, 30, 5, 34, 32, 32) and not ask(lib, 1500, 30, 5, 34, 32, 32)   # one range or two
    assert ask(lib, 8343, 10, 5, 10, 32, 32) and not ask(lib, 8343, 10, 5, 10, 32, 32, 1)  # conversions weigh more
    for units in range(1, 400, 7):
        for chunks in range(1, 300, 13):
            x = lib.cuts(units, chunks)
            assert 1 <= x <= max(1, chunks // 2) and x <= 64 and (x == 1 or (units * x <= lib.most(0) == 256 and units <= lib.most(1)))


SHAPES = [(2100, 30, 5, 34, 32, 32),      # 160 units of 64 rows, one range each; 96 of 128 in two: fp32 partial results
          (804, 30, 5, 30, 40, 40),       # in three
          (3719, 17, 5, 16, 32, 32),      # two ranges; four
          (60, 30, 7, 30, 64, 8)]         # one; one


def inputs(P, W, N, G, H, KV, seed):
    T, rng = 1 + (W + G) * (N - 1), np.random.default_rng(seed)

    def f(*shape):
        return wl.f32_to_bf16_bits(rng.standard_normal(size=shape, dtype=np.float32))
    return dict(q=f(T, H, 128), k_cache=f(KV, P, 128), v_cache=f(KV, P, 128), step_k=f(T, KV, 128), step_v=f(T, KV, 128))


def error(out, want):
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "P%d-W%d-%d/%d" % (s[0], s[1], s[4], s[5]))
def test_every_entry_point_agrees_and_none_is_further_off(shape, override, lib):
    print("case", shape, flush=True)
    P, W, N, G, H, KV = shape
    assert ask(lib, *shape)
    x = inputs(*shape, seed=P)
    dev = {k: binding.bf16_tensor(v) for k, v in x.items()}
    args = (dev["step_k"], dev["step_v"], P, W, N, G, H, KV, 128)

    def new():
        return torch.full(dev["q"].shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    want = orc.step_attention(x["q"], x["k_cache"], x["v_cache"], x["step_k"], x["step_v"], P, W, N, G, H, KV, 128)
    out = binding.la_step_attention(dev["q"], dev["k_cache"], dev["v_cache"], *args, new())
    err = error(out, want)
    # the same bits without an allocation, with room behind the prefix, and from pages
    assert torch.equal(out, binding.la_step_attention_noalloc(dev["q"], dev["k_cache"], dev["v_cache"], *args, new()))
    room = [torch.cat([dev[k], torch.full((KV, 70, 128), float("nan"), dtype=torch.bfloat16, device="cuda")], 1) for k in ("k_cache", "v_cache")]
    assert torch.equal(out, binding.la_step_attention_cap(dev["q"], *room, *args, new()))
    n = -(-P // 64)
    table = torch.randperm(n + 3, device="cuda")[:n]
    pages = []
    for k in ("k_cache", "v_cache"):
        padded = torch.full((KV, n * 64, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        padded[:, :P] = dev[k]
        pool = torch.full((n + 3, KV, 64, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        pool[table] = padded.view(KV, n, 64, 128).transpose(0, 1)
        pages.append(pool)
    assert torch.equal(out, binding.la_step_attention_paged(dev["q"], *pages, table.int(), *args, new()))
    # groups spread over XCDs are computed again
    override("force_recompute", "1")
    error(binding.la_step_attention(dev["q"], dev["k_cache"], dev["v_cache"], *args, new()), want)
    override("force_recompute", None)
    # against 64 bits it is no further off than 64-row workgroups
    override("attn_plan", "2,4,0,4,64")
    assert err <= error(binding.la_step_attention(dev["q"], dev["k_cache"], dev["v_cache"], *args, new()), want)


@pytest.mark.gpu
def test_quantised_cache(lib, override):
    P, W, N, G, H, KV = shape = (1500, 30, 5, 30, 40, 40)
    assert ask(lib, *shape, codes=1)
    T, gen = 1 + (W + G) * (N - 1), torch.Generator(device="cuda").manual_seed(5)

    def codes(*s):
        return torch.randn(s, device="cuda", generator=gen).mul_(112).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    q = torch.randn(T, H, 128, device="cuda", generator=gen).bfloat16()
    kc, vc, sk, sv = codes(KV, P, 128), codes(KV, P, 128), codes(T, KV, 128), codes(T, KV, 128)
    scale = torch.full((2, KV), 4 / 448, device="cuda") * (0.75 + 0.5 * torch.rand(2, KV, device="cuda", generator=gen))
    outs = []
    for plan in (None, "2,4,0,4,64"):
        override("attn_plan", plan)
        outs.append(torch.full_like(q, float("nan")))
        binding.la_step_attention_fp8kv(q, kc, vc, sk, sv, scale[0], scale[1], P, W, N, G, H, KV, 128, outs[-1])
    want = orc.step_attention_fp8kv(binding.bf16_bits(q), *(t.cpu().numpy() for t in (kc, vc, sk, sv)), scale[0].cpu().numpy(),
                                    scale[1].cpu().numpy(), P, W, N, G, H, KV, 128)
    assert error(outs[0], want) <= error(outs[1], want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES[:2], ids=lambda s: "P%d-W%d-%d/%d" % (s[0], s[1], s[4], s[5]))
def test_captured_with_nothing_reserved(shape, override):
    """64-row workgroups need no workspace for a step whose keys are one range, so it can be captured with nothing reserved;
    a graph of it has the eager call's bits all the same."""
    print("case", shape, flush=True)
    P, W, N, G, H, KV = shape
    dev = {k: binding.bf16_tensor(v) for k, v in inputs(*shape, seed=3).items()}
    out = torch.full(dev["q"].shape, float("nan"), dtype=torch.bfloat16, device="cuda")

    def call(entry=binding.la_step_attention):
        entry(dev["q"], dev["k_cache"], dev["v_cache"], dev["step_k"], dev["step_v"], P, W, N, G, H, KV, 128, out)

    def result(*entry):
        out.fill_(float("nan"))
        call(*entry)
        torch.cuda.synchronize()
        return out.clone()
    binding.la_select_workspace(11)
    want = result()                          # (kernels loaded ahead of the capture)
    assert torch.equal(want, result(binding.la_step_attention_noalloc))
    override("attn_plan", "2,4,0,4,64")
    assert not torch.equal(want, result())
    override("attn_plan", None)
    torch.cuda.synchronize()
    binding.la_shutdown()
    binding.la_select_workspace(12)
    try:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            assert torch.equal(result(), want)      # (the workspace reserved in the capture, used outside it)
    finally:
        binding.la_select_workspace(0)
