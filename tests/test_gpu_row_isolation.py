"""A row whose scores are not finite leaves every other row of the step, and every other step of the launch,
what it was, in every kernel: rows share tiles, operands of the matrix cores and workgroups, but no sum."""
import numpy as np
import pytest
import torch

from paper_2402_02057_amd import binding, workloads as wl
from test_gpu_batch import make_seq

pytestmark = pytest.mark.gpu
PAGE = 64


def run_single(steps, W, N, G, H, KV, d):
    s = steps[0]
    binding.la_step_attention(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], s["P"], W, N, G, H, KV, d, s["out"])


def run_rope(steps, W, N, G, H, KV, d):
    s = steps[0]
    cos, sin = [torch.from_numpy(t).cuda() for t in wl.rope_tables(s["P"] + W + N, d)]
    binding.la_step_attention_rope(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], cos, sin, s["P"], W, N, G, H, KV, d,
                                   s["out"], rotate_keys=True)


def run_rows(steps, W, N, G, H, KV, d):
    s = steps[0]
    ids = torch.arange(s["q"].shape[0], dtype=torch.int32, device="cuda")
    binding.la_step_attention_rows(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], ids, s["P"], W, N, G, H, KV, d, s["out"])


def run_fp8(steps, W, N, G, H, KV, d):
    s = steps[0]
    one = torch.ones(KV, dtype=torch.float32, device="cuda")
    codes = [s[k].to(torch.float8_e4m3fn).view(torch.uint8) for k in ("k_cache", "v_cache", "step_k", "step_v")]
    binding.la_step_attention_fp8kv(s["q"], *codes, one, one, s["P"], W, N, G, H, KV, d, s["out"])


def run_batch(steps, W, N, G, H, KV, d):
    assert len(steps) > 1                   # (one alone takes the kernels of the calls above)
    binding.la_step_attention_batch(steps, W, N, G, H, KV, d)


def paged(steps, KV, d):
    """The steps' caches in one pool of pages, back to front; NaN wherever nothing was put."""
    used = [-(-s["P"] // PAGE) for s in steps]
    pools = [torch.full((sum(used), KV, PAGE, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    order, tables, at = list(reversed(range(sum(used)))), [], 0
    for s, n in zip(steps, used):
        tables.append(torch.tensor(order[at:at + n], dtype=torch.int32, device="cuda"))
        for i, page in enumerate(order[at:at + n]):
            for pool, cache in zip(pools, (s["k_cache"], s["v_cache"])):
                rows = cache[:, i * PAGE:(i + 1) * PAGE]
                pool[page, :, :rows.shape[1]] = rows
        at += n
    return pools, tables


def run_paged(steps, W, N, G, H, KV, d):
    s = steps[0]
    (kp, vp), (table,) = paged([s], KV, d)
    binding.la_step_attention_paged(s["q"], kp, vp, table, s["step_k"], s["step_v"], s["P"], W, N, G, H, KV, d, s["out"])


def run_batch_paged(steps, W, N, G, H, KV, d):
    (kp, vp), tables = paged(steps, KV, d)
    binding.la_step_attention_batch_paged([dict(q=s["q"], block_table=t, step_k=s["step_k"], step_v=s["step_v"], out=s["out"], P=s["P"])
                                           for s, t in zip(steps, tables)], kp, vp, W, N, G, H, KV, d)


# (prefixes: of the step that is spoilt, and of one beside it in the launch; what the planner makes of the batches
# is asserted in test_launch_plan.py)
@pytest.mark.parametrize("run,hook,prefixes,H,KV,d", [
    (run_single, ("attn_rowtile", "1"), (300,), 4, 4, 128),
    (run_single, ("attn_rowtile", "0"), (300,), 4, 4, 128),
    (run_single, ("attn_rowtile", "0"), (2100,), 8, 2, 128),
    (run_single, ("attn_rowtile", "0"), (300,), 4, 2, 64),
    (run_single, None, (300,), 4, 1, 128),
    (run_single, None, (4000,), 4, 1, 128),
    (run_paged, ("attn_rowtile", "1"), (300,), 4, 4, 128),
    (run_paged, ("attn_rowtile", "0"), (2100,), 8, 2, 128),
    (run_rope, ("attn_rowtile", "1"), (300,), 4, 4, 128),
    (run_rope, ("attn_rowtile", "0"), (2100,), 8, 2, 128),
    (run_rows, None, (300,), 4, 2, 128),
    (run_fp8, None, (300,), 4, 4, 128),
    (run_batch, ("batch_plan", "2"), (300, 200), 8, 2, 128),         # 64 rows, uncut
    (run_batch, ("batch_plan", "2"), (4000, 300), 32, 8, 128),       # four ranges
    (run_batch, ("batch_plan", "4"), (300, 200), 4, 1, 128),         # 128 rows, uncut
    (run_batch, ("batch_plan", "4"), (4000, 300), 32, 8, 128),       # nine ranges
    (run_batch, ("batch_plan", "8"), (300, 200), 4, 1, 128),         # pipelined, uncut
    (run_batch, ("batch_plan", "8"), (4000, 300), 4, 1, 128),        # ten ranges
    (run_batch, None, (300, 200), 4, 2, 64),
    (run_batch_paged, ("batch_plan", "4"), (4000, 300), 32, 8, 128),
    (run_batch_paged, ("batch_plan", "8"), (4000, 300), 4, 1, 128),
])
def test_rows_that_are_not_finite(override, run, hook, prefixes, H, KV, d):
    print("case", run.__name__, hook, dict(prefixes=prefixes, H=H, KV=KV, d=d), flush=True)
    if hook:
        override(*hook)
    W, N, G = 10, 5, 10
    T = 1 + (W + G) * (N - 1)
    rng = np.random.default_rng(prefixes[0] + H)
    steps = [make_seq(rng, P, T, H, KV, d)[1] for P in prefixes]
    s = steps[0]
    run(steps, W, N, G, H, KV, d)
    want, *beside = [x["out"].float().clone() for x in steps]
    assert all(torch.isfinite(x).all() for x in [want] + beside)
    spoilt = torch.zeros(T, H, dtype=torch.bool, device="cuda")
    for t, h, value in ((3, 0, float("nan")), (40, H - 1, float("inf")), (T - 2, 1, float("nan"))):
        s["q"][t, h] = value
        spoilt[t, h] = True
    s["q"][22, 0, 7] = float("inf")     # infinite scores of both signs, none of them NaN
    spoilt[22, 0] = True
    if run is not run_fp8:          # a key that only the last row sees
        s["step_k"][T - 1] = float("nan")
        spoilt[T - 1] = True
    for x in steps:
        x["out"].fill_(0.5)
    run(steps, W, N, G, H, KV, d)
    got = s["out"].float()
    assert torch.isnan(got[spoilt]).all()
    assert torch.equal(got[~spoilt], want[~spoilt])
    assert all(torch.equal(x["out"].float(), w) for x, w in zip(steps[1:], beside))
