"""Steps alone whose keys are cut into ranges, with any number of row blocks: the ranges of a row block on one XCD (the
mapping of csrc/la_batch_plan.h, on the CPU), and on the GPU no group computed again and none further off."""
import numpy as np
import pytest
import torch

from oracle import la_oracle as orc
from paper_2402_02057_amd import binding, workloads as wl
from step_cases import codes_inputs, error, every_tile_differs, inputs, label, new_like, planner

SHIM = """
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
    lib = planner(tmp_path, SHIM)
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

    def fewer(units, rows, d):                          # numbers of chunks at which a step that always had bf16 takes fewer in fp32
        return [c for c in range(1, 1000) if lib.ranges(units, c, rows, d, 0) < 0]
    for units in (1, 3, 8):
        assert fewer(units, 64, 128) == [53, 57, 59, 61, 63] + list(range(65, 73))
        assert fewer(units, 32, 128) == [59, 63] + list(range(65, 71))
        assert fewer(units, 64, 64) == fewer(units, 32, 64) == \
            list(range(33, 50, 2)) + list(range(51, 91)) + list(range(97, 111)) + list(range(129, 133))
    for units in range(9, 130):
        assert fewer(units, 64, 128) == fewer(units, 32, 128) == [] and fewer(units, 64, 64) == ([33] if units <= 16 else [])


SHAPES = [(700, 5, 4, 5, 4, 4, 128),       # 4 row blocks of 32 rows, 5 ranges each
          (2500, 20, 5, 20, 4, 4, 128),    # 12 of 64 rows, 16
          (3000, 10, 5, 10, 10, 10, 128),  # 20, 10
          (900, 5, 4, 5, 4, 4, 64),
          (2500, 20, 5, 20, 4, 4, 64),
          (300, 15, 5, 15, 50, 50, 128)]   # 100, 2
FEWER = [(4096, 15, 5, 15, 4, 4, 128),     # 8 row blocks: 11 ranges in fp32, 32 in bf16 before
         (3580, 3, 4, 1, 32, 8, 128),      # 8 of 64 rows, 57 chunks: 10 in fp32, 28 in bf16 before
         (4096, 15, 5, 15, 4, 4, 64),
         (4096, 15, 5, 15, 8, 1, 128),     # 16 of 64 rows, 8 of 128 before
         (4096, 16, 5, 15, 16, 2, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=label)
def test_every_entry_point_agrees_and_none_is_further_off(shape, override):
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    T, x = 1 + (W + G) * (N - 1), inputs(shape, P)
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
    # groups spread over XCDs are computed again, over all keys and without partial results: none here is, and that is no nearer
    override("force_recompute", "1")
    again = binding.la_step_attention(q, *cache, *args, new_like(q))
    assert every_tile_differs(out, again, KV) and err <= error(again, want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FEWER, ids=label)
def test_fewer_ranges_are_no_further_off_than_all(shape, override):
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    x = list(inputs(shape, P).values())
    dev = [binding.bf16_tensor(v) for v in x]
    want = orc.step_attention(*x, P, W, N, G, H, KV, d)
    out = binding.la_step_attention(*dev, P, W, N, G, H, KV, d, new_like(dev[0]))
    assert torch.equal(out, binding.la_step_attention_noalloc(*dev, P, W, N, G, H, KV, d, new_like(dev[0])))
    rows = len(x[0]) * H // KV
    override("attn_plan", "4,2,0,4,64" if rows > 480 else "1,2,0,4,64" if rows <= 32 else "2,4,0,4,64" if d == 128 else "2,2,0,4,64")
    before = binding.la_step_attention(*dev, P, W, N, G, H, KV, d, new_like(dev[0]))
    assert every_tile_differs(out, before, KV) and error(out, want) <= error(before, want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES[:5:2], ids=label)
def test_quantised_cache(shape, override):
    print("case", shape, flush=True)
    q, codes, scale = codes_inputs(shape, shape[0])
    want = orc.step_attention_fp8kv(binding.bf16_bits(q), *(t.cpu().numpy() for t in codes), scale[0].cpu().numpy(),
                                    scale[1].cpu().numpy(), *shape)
    outs = []
    for again in (None, "1"):
        override("force_recompute", again)
        outs.append(binding.la_step_attention_fp8kv(q, *codes, scale[0], scale[1], *shape, new_like(q)))
    assert every_tile_differs(*outs, shape[5]) and error(outs[0], want) <= error(outs[1], want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES + FEWER[:3], ids=label)
def test_true_subsets_of_the_rows(shape, override):
    """Some of the rows, in another order: none is computed again over all keys."""
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    x, rng = inputs(shape, P), np.random.default_rng(P + 1)
    T = len(x["q"])
    ids = np.concatenate([[0], 1 + rng.permutation(T - 1)[:T * 3 // 4]])
    q, sk, sv = (binding.bf16_tensor(x[k][ids]) for k in ("q", "step_k", "step_v"))
    kc, vc, on_gpu = binding.bf16_tensor(x["k_cache"]), binding.bf16_tensor(x["v_cache"]), torch.from_numpy(ids.astype(np.int32)).cuda()
    want = orc.step_attention_rows(x["q"][ids], x["k_cache"], x["v_cache"], x["step_k"][ids], x["step_v"][ids], ids, P, W, N, G, H, KV, d)

    def run():
        return binding.la_step_attention_rows(q, kc, vc, sk, sv, on_gpu, P, W, N, G, H, KV, d, new_like(q))
    out = run()
    error(out, want)
    override("force_recompute", "1")
    assert every_tile_differs(out, run(), KV)


@pytest.mark.gpu
@pytest.mark.parametrize("interleaved", [False, True])
@pytest.mark.parametrize("shape", SHAPES + FEWER[:3], ids=label)
def test_rotations(shape, interleaved, override):
    """Query rows and step keys rotated inside the attention have the bits of both rotated in memory first."""
    print("case", shape, flush=True)
    P, W, N, G, H, KV, d = shape
    x = inputs(shape, P)
    dev = {k: binding.bf16_tensor(v) for k, v in x.items()}
    cos, sin = wl.rope_tables(P + W + N, d)
    tables = torch.from_numpy(cos).cuda(), torch.from_numpy(sin).cuda()
    sizes = P, W, N, G, H, KV, d
    override("attn_rowtile", "0")
    q2, k2 = dev["q"].clone(), dev["step_k"].clone()
    binding.la_step_rope(q2, k2, *tables, *sizes, interleaved)
    two = binding.la_step_attention(q2, dev["k_cache"], dev["v_cache"], k2, dev["step_v"], *sizes, new_like(q2))

    def run():
        return binding.la_step_attention_rope(dev["q"], dev["k_cache"], dev["v_cache"], dev["step_k"], dev["step_v"], *tables, *sizes,
                                              new_like(q2), interleaved, rotate_keys=True)
    out = run()
    assert torch.equal(out, two)
    rq, rk = orc.step_rope(orc.bf16_to_f64(x["q"]), orc.bf16_to_f64(x["step_k"]), cos, sin, P, W, N, G, interleaved)
    error(out, orc.step_attention(wl.f32_to_bf16_bits(rq.astype(np.float32)), x["k_cache"], x["v_cache"],
                                  wl.f32_to_bf16_bits(rk.astype(np.float32)), x["step_v"], *sizes))
    override("force_recompute", "1")
    assert every_tile_differs(out, run(), KV)
