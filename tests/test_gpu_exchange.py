"""Which wave adds up the ranges of a step's keys (csrc/la_attention.hip) does not show in the results: the one that is
to, which waits for the others, or, where it has stopped waiting, the last one to arrive."""
import pytest
import torch

from paper_2402_02057_amd import binding
from tests.step_cases import codes_inputs, label, new_like

pytestmark = pytest.mark.gpu

# P, W, N, G, heads, KV heads, head_dim and the decomposition (None: the library's): 2 to 8 and 32 ranges, more and fewer
# than the eight, four or two waves of a workgroup; one and two slices a wave; a row block of one tile; fp32 results
CASES = [((1024, 15, 5, 15, 32, 32, 128), None), ((2048, 10, 5, 10, 40, 40, 128), "2,4,3,4,64"), ((700, 9, 4, 5, 8, 8, 128), "2,4,2,4,64"),
         ((700, 9, 4, 5, 8, 8, 128), "2,4,5,4,64"), ((700, 9, 4, 5, 8, 8, 128), "1,2,6,4,64"), ((194, 7, 3, 7, 20, 20, 128), None), ((2100, 30, 5, 34, 32, 32, 128), None),
         ((900, 9, 4, 5, 8, 8, 64), "2,2,7,4,64"),
         ((2100, 10, 5, 10, 40, 40, 128), "4,2,6,4,64"), ((4096, 7, 5, 7, 64, 8, 128), "4,2,8,4,64"), ((4096, 15, 5, 15, 4, 4, 128), "2,4,32,4,64"),
         ((4096, 15, 5, 15, 4, 4, 128), None), ((4096, 3, 4, 2, 4, 4, 128), None), ((4096, 15, 5, 15, 4, 4, 64), None), ((3000, 3, 4, 2, 8, 8, 64), None)]


@pytest.mark.parametrize("kind", ["packed", "paged", "fp8"])
@pytest.mark.parametrize("shape,plan", CASES, ids=["%s-%s" % (label(s), (p or "own").replace(",", "_")) for s, p in CASES])
def test_whoever_adds_up(shape, plan, kind, override):
    P, W, N, G, H, KV, d = shape
    gen = torch.Generator(device="cuda").manual_seed(11)
    if kind == "fp8":
        q, (kc, vc, sk, sv), scale = codes_inputs(shape, 11)
    else:
        pages = -(-P // 64)
        cache = (pages, KV, 64, d) if kind == "paged" else (KV, P, d)
        T = 1 + (W + G) * (N - 1)
        q, kc, vc, sk, sv = (torch.randn(s, device="cuda", generator=gen).bfloat16() for s in ((T, H, d), cache, cache, (T, KV, d), (T, KV, d)))
        table = torch.randperm(pages, device="cuda", generator=gen).int()

    def run():
        out = new_like(q)
        if kind == "fp8":
            binding.la_step_attention_fp8kv(q, kc, vc, sk, sv, scale[0], scale[1], P, W, N, G, H, KV, d, out)
        elif kind == "paged":
            binding.la_step_attention_paged(q, kc, vc, table, sk, sv, P, W, N, G, H, KV, d, out)
        else:
            binding.la_step_attention(q, kc, vc, sk, sv, P, W, N, G, H, KV, d, out)
        return out.view(torch.int16)
    override("attn_rowtile", "0")
    if plan:
        override("attn_plan", plan)
    override("exchange_looks", "0")
    last = run()
    for looks in ("1", "2", None):     # (with one look most leave; the tickets are clean again for each next call)
        override("exchange_looks", looks)
        for _ in range(5):
            assert torch.equal(run(), last), looks
