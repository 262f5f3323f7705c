"""GPU parity of the pipelined batch kernel (256-row workgroups), forced by the batch_plan hook: against the
oracle, and for what the oracle does not say against the staged kernel."""
import numpy as np
import pytest
import torch

from oracle import la_oracle as orc
from paper_2402_02057_amd import binding, workloads as wl
from test_gpu_batch import bits, make_seq, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefixes,W,N,G,H,KV", [
    ([0, 1, 63, 64, 65], 10, 5, 10, 8, 2),              # no prefix, and around the edge of a chunk; 11 tiles in blocks of 6 and 5
    ([128, 127, 320, 383], 15, 5, 15, 4, 1),            # walks of two to six full chunks; two row blocks of eight tiles
    ([200, 500], 4, 7, 4, 6, 2),                        # a group of three: 5 tiles, the last with 19 rows
    ([700, 64], 3, 3, 12, 4, 1),                        # four tiles of which the last has 28 rows
    ([1500] * 3, 30, 3, 30, 8, 8),                      # one query head per KV head: four tiles, one row in the last block's last
    ([9000, 40, 7000], 15, 5, 15, 4, 1),                # cut into many ranges, beside a step that is not
    ([6000, 3000, 1500], 20, 5, 3, 16, 2),              # ranges that end among the step's own keys
    ([300] * 17 + [90], 10, 5, 10, 4, 1),               # more than one launch
])
def test_pipelined_against_the_oracle(override, prefixes, W, N, G, H, KV):
    print("case", dict(prefixes=prefixes, W=W, N=N, G=G, H=H, KV=KV), flush=True)
    override("batch_plan", "8")
    order = np.argsort(prefixes, kind="stable")
    run_batch(prefixes, W, N, G, H, KV, 128, seed=sum(prefixes) + W, check_oracle={int(order[0]), int(order[-1])})


@pytest.mark.parametrize("prefixes,page", [([4700, 100, 64, 0], 64), ([9000, 2049], 128)])   # more than 64 pages: the entries are fetched again
def test_pages(override, prefixes, page):
    """The bits of the packed batch, whose result the test above compares with the oracle."""
    override("batch_plan", "8")
    print("case", dict(prefixes=prefixes, page=page), flush=True)
    W, N, G, H, KV, d = 15, 5, 15, 8, 2, 128
    rng = np.random.default_rng(page)
    T = 1 + (W + G) * (N - 1)
    seqs = [make_seq(rng, P, T, H, KV, d) for P in prefixes]
    used = [-(-P // page) for P in prefixes]
    perm = rng.permutation(sum(used) + 2).astype(np.int32)
    kp = np.full((len(perm), KV, page, d), 0x7FC0, dtype=np.uint16)     # NaN wherever nothing was put
    vp = kp.copy()
    descs, at = [], 0
    binding.la_step_attention_batch([dev for _, dev in seqs], W, N, G, H, KV, d)
    for (x, dev), P, n in zip(seqs, prefixes, used):
        table = perm[at:at + n]
        at += n
        for i in range(n):
            lo, hi = i * page, min(P, (i + 1) * page)
            kp[table[i], :, :hi - lo] = x["k_cache"][:, lo:hi]
            vp[table[i], :, :hi - lo] = x["v_cache"][:, lo:hi]
        descs.append(dict(q=dev["q"], step_k=dev["step_k"], step_v=dev["step_v"], P=P, out=torch.empty_like(dev["out"]),
                          block_table=torch.from_numpy(np.ascontiguousarray(table)).cuda() if n else None))
    binding.la_step_attention_batch_paged(descs, binding.bf16_tensor(kp), binding.bf16_tensor(vp), W, N, G, H, KV, d)
    torch.cuda.synchronize()
    for (_, dev), desc in zip(seqs, descs):
        assert torch.equal(dev["out"].view(torch.int16), desc["out"].view(torch.int16))


def test_what_nobody_sees_is_not_read(override):
    """Infinite values in the last candidates, whose blocks the first tiles pass over: the rows that come out
    finite are those of the staged kernel, and equal to its to bf16 rounding of both (2 ** -7 of a value, and as much of 1)."""
    W, N, G, H, KV, d = 20, 5, 20, 8, 2, 128
    T = 1 + (W + G) * (N - 1)
    rng = np.random.default_rng(5)
    seqs = [make_seq(rng, P, T, H, KV, d)[1] for P in (100, 700)]
    for s in seqs:
        s["step_v"][T - 2 * (N - 1):] = float("inf")
    outs = []
    for plan in ("4", "8"):
        override("batch_plan", plan)
        binding.la_step_attention_batch(seqs, W, N, G, H, KV, d)
        torch.cuda.synchronize()
        outs.append([s["out"].float().clone() for s in seqs])
    for a, b in zip(*outs):
        assert torch.equal(torch.isfinite(a), torch.isfinite(b)) and torch.isfinite(a).any() and not torch.isfinite(a).all()
        ok = torch.isfinite(a)
        assert ((a - b).abs()[ok] <= (a.abs()[ok] + 1) * 2.0 ** -7).all()


def test_captured_and_replayed(override):
    """A cut launch is two kernels over one workspace: recorded after an uncut eager batch, replayed with eager
    batches between."""
    override("batch_plan", "8")
    W, N, G, H, KV, d = 15, 5, 15, 8, 2, 128
    T = 1 + (W + G) * (N - 1)
    rng = np.random.default_rng(6)
    small, large = [[make_seq(rng, P, T, H, KV, d)[1] for P in ps] for ps in ((100, 90), (5000, 3000, 200))]
    binding.la_step_attention_batch(small, W, N, G, H, KV, d)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.la_step_attention_batch(large, W, N, G, H, KV, d)
    binding.la_step_attention_batch(large, W, N, G, H, KV, d)
    torch.cuda.synchronize()
    want = [s["out"].clone() for s in large]
    for _ in range(3):
        for s in large:
            s["out"].fill_(float("nan"))
        binding.la_step_attention_batch(small, W, N, G, H, KV, d)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(s["out"].view(torch.int16), w.view(torch.int16)) for s, w in zip(large, want))
