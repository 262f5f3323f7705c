"""Row subsets at the ends of what the mask's line numbers and the staged ids take."""
import numpy as np
import pytest

from oracle import la_oracle as orc
from test_gpu_rows import TOL, bits, run_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,W,N,G,n", [
    (40, 0, 5, 9, 30),          # no window: candidates alone
    (40, 9, 5, 0, 30),          # no candidates
    (0, 1, 2, 1, 3),            # one column, one level, one token
    (64, 140, 5, 140, 1024),    # as many rows as are taken, of 1121
    (64, 300, 2, 700, 513),     # many lines of one row each
    (130, 2, 30, 2, 64),        # few long lines
])
def test_subsets(P, W, N, G, n):
    print("case", dict(P=P, W=W, N=N, G=G, rows=n), flush=True)
    rng = np.random.default_rng(W * 1000 + n)
    T, H, KV, d = 1 + (W + G) * (N - 1), 2, 1, 128
    x = dict(q=bits(rng, (T, H, d)), k_cache=bits(rng, (KV, P, d)), v_cache=bits(rng, (KV, P, d)),
             step_k=bits(rng, (T, KV, d)), step_v=bits(rng, (T, KV, d)))
    ids = rng.permutation(T)[:n]
    if 0 not in ids:
        ids[-1] = 0             # (a row that sees no key at all has no softmax)
    got = run_rows(x, ids, P, W, N, G, H, KV, d)
    want = orc.step_attention_rows(x["q"][ids], x["k_cache"], x["v_cache"], x["step_k"][ids], x["step_v"][ids], ids, P, W, N, G, H, KV, d)
    assert np.abs(got - want).max() <= TOL
