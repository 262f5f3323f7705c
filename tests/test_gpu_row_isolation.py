"""A row whose scores are not finite leaves every other row of the step what it was, in every kernel: rows
share tiles, operands of the matrix cores and workgroups, but no sum."""
import numpy as np
import pytest
import torch

from paper_2402_02057_amd import binding
from test_gpu_batch import make_seq

pytestmark = pytest.mark.gpu


def run_single(s, P, W, N, G, H, KV, d):
    binding.la_step_attention(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], P, W, N, G, H, KV, d, s["out"])


def run_rows(s, P, W, N, G, H, KV, d):
    ids = torch.arange(s["q"].shape[0], dtype=torch.int32, device="cuda")
    binding.la_step_attention_rows(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], ids, P, W, N, G, H, KV, d, s["out"])


def run_batch(s, P, W, N, G, H, KV, d):
    binding.la_step_attention_batch([s], W, N, G, H, KV, d)


def run_fp8(s, P, W, N, G, H, KV, d):
    one = torch.ones(KV, dtype=torch.float32, device="cuda")
    codes = [s[k].to(torch.float8_e4m3fn).view(torch.uint8) for k in ("k_cache", "v_cache", "step_k", "step_v")]
    binding.la_step_attention_fp8kv(s["q"], *codes, one, one, P, W, N, G, H, KV, d, s["out"])


@pytest.mark.parametrize("run,hook,P,H,KV,d", [
    (run_single, ("attn_rowtile", "1"), 300, 4, 4, 128),
    (run_single, ("attn_rowtile", "0"), 300, 4, 4, 128),
    (run_single, ("attn_rowtile", "0"), 2100, 8, 2, 128),
    (run_single, ("attn_rowtile", "0"), 300, 4, 2, 64),
    (run_rows, None, 300, 4, 2, 128),
    (run_fp8, None, 300, 4, 4, 128),
    (run_batch, ("batch_plan", "2"), 300, 4, 1, 128),
    (run_batch, ("batch_plan", "4"), 300, 4, 1, 128),
    (run_batch, ("batch_plan", "8"), 300, 4, 1, 128),
    (run_batch, ("batch_plan", "8"), 4000, 4, 1, 128),
])
def test_rows_that_are_not_finite(override, run, hook, P, H, KV, d):
    print("case", run.__name__, hook, dict(P=P, H=H, KV=KV, d=d), flush=True)
    if hook:
        override(*hook)
    W, N, G = 10, 5, 10
    T = 1 + (W + G) * (N - 1)
    s = make_seq(np.random.default_rng(P + H), P, T, H, KV, d)[1]
    run(s, P, W, N, G, H, KV, d)
    want = s["out"].float().clone()
    assert torch.isfinite(want).all()
    spoilt = torch.zeros(T, H, dtype=torch.bool, device="cuda")
    for t, h, value in ((3, 0, float("nan")), (40, H - 1, float("inf")), (T - 2, 1, float("nan"))):
        s["q"][t, h] = value
        spoilt[t, h] = True
    s["q"][22, 0, 7] = float("inf")     # infinite scores of both signs, none of them NaN
    spoilt[22, 0] = True
    if run is not run_fp8:          # a key that only the last row sees
        s["step_k"][T - 1] = float("nan")
        spoilt[T - 1] = True
    run(s, P, W, N, G, H, KV, d)
    got = s["out"].float()
    assert torch.isnan(got[spoilt]).all()
    assert torch.equal(got[~spoilt], want[~spoilt])
