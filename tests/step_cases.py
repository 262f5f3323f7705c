"""What the tests of single steps' plans (test_step_rows.py, test_step_ranges.py) share."""
import ctypes
import os
import subprocess

import numpy as np
import torch

from paper_2402_02057_amd import buildlib, workloads as wl

TOL = 2e-2


def planner(folder, functions):
    """csrc/la_batch_plan.h with some C functions over it, as a library."""
    (folder / "shim.cpp").write_text('#include "la_batch_plan.h"\n' + functions)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", buildlib.CSRC,
                    str(folder / "shim.cpp"), "-o", str(folder / "shim.so")], check=True)
    return ctypes.CDLL(str(folder / "shim.so"))


def label(shape):
    return "P%d-W%d-%d/%d-d%d" % (shape[0], shape[1], shape[4], shape[5], shape[6])


def inputs(shape, seed):
    P, W, N, G, H, KV, d = shape
    T, rng = 1 + (W + G) * (N - 1), np.random.default_rng(seed)

    def f(*s):
        return wl.f32_to_bf16_bits(rng.standard_normal(size=s, dtype=np.float32))
    return dict(q=f(T, H, d), k_cache=f(KV, P, d), v_cache=f(KV, P, d), step_k=f(T, KV, d), step_v=f(T, KV, d))


def codes_inputs(shape, seed):
    """Rows q in bf16, keys and values as 8-bit floats (cache and step), scales, all on the GPU."""
    P, W, N, G, H, KV, d = shape
    T, gen = 1 + (W + G) * (N - 1), torch.Generator(device="cuda").manual_seed(seed)

    def codes(*s):
        return torch.randn(s, device="cuda", generator=gen).mul_(112).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    q = torch.randn(T, H, d, device="cuda", generator=gen).bfloat16()
    scale = torch.full((2, KV), 4 / 448, device="cuda") * (0.75 + 0.5 * torch.rand(2, KV, device="cuda", generator=gen))
    return q, [codes(KV, P, d), codes(KV, P, d), codes(T, KV, d), codes(T, KV, d)], scale


def new_like(q):
    return torch.full_like(q, float("nan"))


def error(out, want):
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


def every_tile_differs(a, b, kv_heads):
    """Whether no 32-row tile of any KV head has the same bits in both: none came about in the same way."""
    T, heads, _ = a.shape
    rows = (a != b).any(-1).view(T, kv_heads, heads // kv_heads).transpose(0, 1).reshape(kv_heads, -1)
    return all(bool(tile.any(1).all()) for tile in rows.split(32, 1))
