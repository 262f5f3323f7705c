"""Steps alone that take 128-row workgroups: where the rule draws the line (csrc/la_batch_plan.h, on the CPU), and
on the GPU the steps on its other side, cut with fp32 partial results, cut with bf16 ones and whole."""
import pytest
import torch

from oracle import la_oracle as orc
from paper_2402_02057_amd import binding, workloads as wl
from step_cases import codes_inputs, error, every_tile_differs, inputs, label, new_like, planner

SHIM = """
extern "C" int rows128(int chunks, int tiles, int kv_heads, int many, int codes) { return la::step_rows128(chunks, tiles, kv_heads, many, codes); }
extern "C" int cuts(int units, int chunks) { return la::step_cuts(units, chunks); }
extern "C" int ahead(int rows, int head_dim, int blocks, int range) { return la::step_chunks_ahead(rows, head_dim, blocks, range); }
extern "C" int most(int groups) { return groups ? la::kMaxStepGroups : la::kMaxStepWorkgroups; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return planner(tmp_path_factory.mktemp("step_rows"), SHIM)


def ask(lib, P, W, N, G, H, KV, d=128, codes=0):
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
    assert ask(lib, 8343, 10, 5, 10, 32, 32) and not ask(lib, 8343, 10, 5, 10, 32, 32, codes=1)  # conversions weigh more
    for units in range(1, 400, 7):
        for chunks in range(1, 300, 13):
            x = lib.cuts(units, chunks)
            assert 1 <= x <= max(1, chunks // 2) and x <= 64 and (x == 1 or (units * x <= lib.most(0) == 256 and units <= lib.most(1)))


def test_chunks_requested_ahead(lib):
    for rows, d, blocks, chunks, want in ((128, 128, 1, 3, 1), (128, 128, 1, 4, 2), (128, 128, 1, 200, 2), (128, 128, 2, 3, 1), (128, 128, 2, 4, 2),
                                          (128, 128, 2, 31, 2), (128, 128, 2, 32, 4), (32, 128, 1, 1, 2), (32, 128, 1, 200, 2), (64, 64, 3, 16, 2), (64, 64, 3, 17, 3)):
        assert lib.ahead(rows, d, blocks, chunks) == want, (rows, d, blocks, chunks)


SHAPES = [(2100, 30, 5, 34, 32, 32, 128), # 160 units of 64 rows, one range each; 96 of 128 in two: fp32 partial results
          (804, 30, 5, 30, 40, 40, 128),  # in three
          (3719, 17, 5, 16, 32, 32, 128), # two ranges; four
          (60, 30, 7, 30, 64, 8, 128)]    # one; one


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=label)
def test_every_entry_point_agrees_and_none_is_further_off(shape, override, lib):
    print("case", shape, flush=True)
    P, KV = shape[0], shape[5]
    assert ask(lib, *shape)
    x = inputs(shape, P)
    dev = {k: binding.bf16_tensor(v) for k, v in x.items()}
    args = (dev["step_k"], dev["step_v"], *shape)

    def new():
        return new_like(dev["q"])
    want = orc.step_attention(*x.values(), *shape)
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
    # it is another result than 64-row workgroups', and against 64 bits no further off
    override("attn_plan", "2,4,0,4,64")
    rows64 = binding.la_step_attention(dev["q"], dev["k_cache"], dev["v_cache"], *args, new())
    assert every_tile_differs(out, rows64, KV) and err <= error(rows64, want)


@pytest.mark.gpu
def test_quantised_cache(lib, override):
    shape = (1500, 30, 5, 30, 40, 40, 128)
    assert ask(lib, *shape, codes=1)
    q, codes, scale = codes_inputs(shape, 5)
    outs = []
    for plan in (None, "2,4,0,4,64"):
        override("attn_plan", plan)
        outs.append(binding.la_step_attention_fp8kv(q, *codes, scale[0], scale[1], *shape, new_like(q)))
    want = orc.step_attention_fp8kv(binding.bf16_bits(q), *(t.cpu().numpy() for t in codes), scale[0].cpu().numpy(),
                                    scale[1].cpu().numpy(), *shape)
    assert every_tile_differs(*outs, 40) and error(outs[0], want) <= error(outs[1], want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES[:2], ids=label)
def test_captured_with_nothing_reserved(shape, override):
    """64-row workgroups need no workspace for a step whose keys are one range, so it can be captured with nothing reserved;
    a graph of it has the eager call's bits all the same."""
    print("case", shape, flush=True)
    dev = {k: binding.bf16_tensor(v) for k, v in inputs(shape, 3).items()}
    out = new_like(dev["q"])

    def call(entry=binding.la_step_attention):
        entry(dev["q"], dev["k_cache"], dev["v_cache"], dev["step_k"], dev["step_v"], *shape, out)

    def result(*entry):
        out.fill_(float("nan"))
        call(*entry)
        torch.cuda.synchronize()
        return out.clone()
    binding.la_select_workspace(11)
    want = result()                          # (kernels loaded ahead of the capture)
    assert torch.equal(want, result(binding.la_step_attention_noalloc))
    override("attn_plan", "2,4,0,4,64")
    assert every_tile_differs(want, result(), shape[5])
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
