"""The work a user of this framework has it do, as cases that can be timed and compared.

A decoding step of a model is, per layer, one attention call over that layer's KV cache; then one
verification of the step's logits; then one append of the accepted tokens to all layers' caches.
Most cases are such a step, with the layer count of the model they are shaped like, because that
is what the entry points are called for, step after step:

  call    one attention call and one verification on their own
  step    a greedy or sampling step of one sequence: cache in place, in pages, packed with the
          rotary embedding inside the attention, or packed in 8-bit floats
  batch   a step of several sequences with prefixes of their own, one launch per layer
  share   one device's rows of a wide step under lookahead parallelism
  loop    the decoding loop itself on the toy model, host logic and one read per step included

Shapes come from paper_2402_02057_amd/workloads.py and bench.py (the settings the paper reports as
good for its model sizes), the step sizes around them from the ragged sweep and the tests.  Inputs
are made on the GPU from the seed: N(0,1) activations, keys and values; logits with planted
accepted runs.
"""
import random

import numpy as np
import torch

from paper_2402_02057_amd import binding, lookahead, workloads as wl

# heads, KV heads, head_dim, layers, vocabulary
GEOMETRY = {
    "tiny": (4, 4, 64, 8, 512),
    "7b": (32, 32, 128, 32, 32000),
    "13b": (40, 40, 128, 40, 32000),
    "70b": (64, 8, 128, 80, 32000),
    "gqa": (32, 8, 128, 32, 32016),
}
PEAK = float(wl.PLANT_VALUE)


def _case(kind, shape, **more):
    heads, kv_heads, head_dim, layers, vocab = GEOMETRY[shape]
    return dict(dict(kind=kind, heads=heads, kv_heads=kv_heads, head_dim=head_dim, layers=layers, V=vocab), **more)


def _text(lengths):
    return ",".join(str(n) for n in lengths)


def listed():
    tiny, p256, b7, b13, b70 = wl.TINY, wl.LLAMA2_7B_P256, wl.LLAMA2_7B, wl.LLAMA2_13B, wl.LLAMA2_70B

    def of(s):
        return dict(P=s.P, W=s.W, N=s.N, G=s.G)
    return [
        # the smallest use: one layer's attention and one verification, all latency
        dict(_case("call", "tiny", **of(tiny)), layers=1, name="tiny call"),
        # the first steps after a short prompt
        dict(_case("step", "7b", cache="inplace", sampling=False, **of(p256)), name="7b short prompt"),
        # the benchmark's headline step
        dict(_case("step", "7b", cache="inplace", sampling=False, **of(b7)), name="7b step"),
        # the same model with the rotary embedding inside the attention, ragged sizes all over
        dict(_case("step", "7b", cache="rope", sampling=False, P=1533, W=13, N=4, G=9), name="7b rope, odd sizes"),
        # sampling instead of greedy verification, cache in pages as a serving system holds it
        dict(_case("step", "7b", cache="paged", page=64, sampling=True, P=777, W=15, N=5, G=15), name="7b paged sampling"),
        # the middle model
        dict(_case("step", "13b", cache="inplace", sampling=False, **of(b13)), name="13b step"),
        # and with its cache quantised to 8-bit floats
        dict(_case("step", "13b", cache="fp8", sampling=False, **of(b13)), name="13b 8-bit cache"),
        # the large model with grouped queries
        dict(_case("step", "70b", cache="inplace", sampling=False, **of(b70)), name="70b gqa step"),
        # eight sequences of very different lengths side by side, one pool of pages: the largest
        dict(_case("batch", "gqa", cache="paged", page=64, sampling=False, prefixes=_text(wl.ragged_prefix_lengths()),
                   W=15, N=5, G=15), name="ragged batch"),
        # a serving batch of sequences of middling length that sample, packed caches
        dict(_case("batch", "gqa", cache="packed", sampling=True,
                   prefixes=_text([1021 - 37 * i for i in range(16)]), W=10, N=5, G=10), name="sampling batch"),
        # a quarter of a step so wide that it was made for four devices
        dict(_case("share", "7b", P=1024, W=60, N=5, G=60, parts=4, part=1), name="quarter of a wide step"),
        # the loop: window, n-gram pool, verification, append, one read per step
        dict(kind="loop", seqs=1, tokens=96, prompt=24, W=15, N=5, G=15, page=0, temperature=0.0, name="decoding loop"),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def _draw(rng):
    kind = rng.choice(["call", "step", "step", "step", "step", "step", "batch", "batch", "share", "loop"])
    N = rng.choice([3, 4, 5, 5, 5, 6, 7])
    W = rng.choice([3, 5, 7, 10, 13, 15, 15, 20, 30])
    G = rng.choice([W, W, rng.randint(1, W)])
    if kind == "call":
        shape = rng.choice(["tiny", "7b", "70b", "gqa"])
        c = _case("call", shape, P=_log(rng, 16, 8192), W=W, N=N, G=G)
        c["layers"] = 1
        return c
    if kind == "step":
        shape = rng.choice(["tiny", "7b", "7b", "13b", "70b", "gqa"])
        cache = rng.choice(["inplace", "inplace", "paged", "rope", "fp8"])
        c = _case("step", shape, cache=cache, sampling=cache in ("inplace", "paged") and rng.random() < 0.3,
                  P=_log(rng, 32, 16384), W=min(W, 20) if cache == "rope" else W, N=N, G=G)
        if cache == "paged":
            c["page"] = rng.choice([64, 128, 256])
        c["G"] = min(c["G"], c["W"])
        return c
    if kind == "batch":
        shape = rng.choice(["7b", "gqa", "gqa"])
        cache = rng.choice(["packed", "paged"])
        seqs = _log(rng, 2, 32)
        top = _log(rng, 64, 16384)
        c = _case("batch", shape, cache=cache, sampling=rng.random() < 0.3, W=W, N=N, G=G,
                  prefixes=_text([_log(rng, max(1, top // 16), top) for _ in range(seqs)]))
        if cache == "paged":
            c["page"] = rng.choice([64, 128])
        return c
    if kind == "share":
        W = rng.choice([20, 30, 40, 60])
        parts = rng.choice([2, 4, 8])
        return _case("share", rng.choice(["7b", "gqa"]), P=_log(rng, 64, 8192), W=W, N=rng.choice([4, 5]), G=W,
                     parts=parts, part=rng.randrange(parts))
    return dict(kind="loop", seqs=rng.choice([1, 1, 4, 8]), tokens=rng.randint(24, 96), prompt=rng.randint(8, 64), W=W, N=N,
                G=G, page=0, temperature=0.0)


def _prefixes(case):
    return [int(x) for x in case["prefixes"].split(",")] if "prefixes" in case else [case["P"]]


def _rows(case):
    return 1 + (case["W"] + case["G"]) * (case["N"] - 1)


def _state_bytes(case):
    if case["kind"] == "loop":
        return 0
    return case["layers"] * sum(4 * case["kv_heads"] * case["head_dim"] * P for P in _prefixes(case))


def draw(rng):
    most = next(work(c) for c in listed() if c["name"] == "ragged batch")
    while True:
        c = _draw(rng)
        if c["kind"] == "loop":
            if c["seqs"] > 1:
                c["page"] = 64
                c["tokens"] = min(c["tokens"], 48)
            else:
                c["page"] = rng.choice([0, 64])
                c["temperature"] = rng.choice([0.0, 0.0, 1.0])
            return c
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"] and _state_bytes(c) < 12e9:
            return c


# ---- what a pass cannot do without ------------------------------------------------------------

def _visible_pairs(W, N, G):
    n1 = N - 1
    return 1 + sum(2 + j for j in range(W)) + sum(2 + j + l for l in range(1, n1) for j in range(W)) \
        + G * sum(2 + k for k in range(n1))


def work(case):
    W, N, G = case["W"], case["N"], case["G"]
    n1, T = N - 1, _rows(case)
    if case["kind"] == "loop":
        # at least one step per N tokens: the step's rows through one head of 64 and their logits
        steps = -(-case["tokens"] // N) * case["seqs"]
        cached = case["prompt"] + case["tokens"] // 2
        return {"bytes": steps * (T * 64 * 2 * 4 + cached * 64 * 2 * 2 + T * wl.TOY_VOCAB * 4),
                "flops": steps * 4 * 64 * T * cached}
    H, KV, d, L, V = case["heads"], case["kv_heads"], case["head_dim"], case["layers"], case["V"]
    rows = len(lookahead.lp_share(W, N, G, case["parts"], case["part"])) if case["kind"] == "share" else T
    elem = 1 if case.get("cache") == "fp8" else 2
    bytes_ = flops = 0
    for P in _prefixes(case):
        bytes_ += L * (2 * (P + rows) * KV * d * elem + 2 * rows * H * d * 2)
        flops += L * 4 * d * H * (rows * P + _visible_pairs(W, N, G) * rows // T)
        if case["kind"] == "share":
            continue
        if case["kind"] == "call":
            bytes_ += G * n1 * (V * 4 + 8)
        else:
            bytes_ += (1 + W + G * n1) * V * 4
        if case.get("cache") in ("inplace", "paged"):
            bytes_ += L * 2 * 2 * 2 * KV * d * 2        # two rows read and written, in keys and values
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # tokens, counts and appended rows are the same; attention rows are bf16 results of bf16 inputs
    return "exact" if case["kind"] == "loop" else {"rel": 1e-2}


# ---- inputs ------------------------------------------------------------------------------------

class _Inputs:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.host = random.Random(seed)

    def normal(self, *shape, dtype=torch.bfloat16):
        return torch.randn(*shape, dtype=dtype, device="cuda", generator=self.gen)

    def uniform(self, *shape):
        return torch.rand(*shape, device="cuda", generator=self.gen)

    def codes(self, *shape):
        """8-bit floats of N(0,1) values under the scale 4/448 (their largest magnitude is about 4)."""
        x = torch.empty(shape, dtype=torch.uint8, device="cuda")
        for part in x.view(-1).split(1 << 26):
            v = torch.randn(part.shape, device="cuda", generator=self.gen).mul_(448.0 / 4.0).clamp_(-448.0, 448.0)
            part.copy_(v.to(torch.float8_e4m3fn).view(torch.uint8))
        return x


def _ints(*shape):
    return torch.zeros(shape, dtype=torch.int32, device="cuda")


def _plant(x, V, W, N, G):
    """Logits of one sequence's step with candidate runs of every length, as a model that agrees
    with some of its candidates gives: {cur, look, cand, tokens}."""
    n1, host = N - 1, x.host
    cur, look, cand = x.normal(V, dtype=torch.float32), x.normal(W, V, dtype=torch.float32), x.normal(G, n1, V, dtype=torch.float32)
    first, shift = host.randrange(V), host.randrange(N)
    cur[first] = PEAK
    rows, cols, toks = [], [], []
    for g in range(G):
        length = (g + shift) % N
        t = [host.randrange(V) for _ in range(n1)]
        t[0] = first if length else (first + 1 + host.randrange(V - 1)) % V
        for slot in range(1, n1 + 1):        # slot's token is judged by the row before it; the last row is the bonus row
            rows.append(g * n1 + slot - 1)
            cols.append(t[slot] if slot < length and slot < n1 else host.randrange(V))
        toks.append(t)
    if G:
        cand.view(G * n1, V)[torch.tensor(rows, device="cuda"), torch.tensor(cols, device="cuda")] = PEAK
    look[torch.arange(W, device="cuda"), torch.tensor([host.randrange(V) for _ in range(W)], device="cuda")] = PEAK
    return dict(cur=cur, look=look, cand=cand, toks=toks, tokens=torch.tensor(toks, dtype=torch.int32, device="cuda").view(G, n1),
                u_test=x.uniform(n1, G), u_final=x.uniform(1))


def _verify_desc(v):
    return dict(logits_cur=v["cur"], logits_look=v["look"], logits_cand=v["cand"], cand_tokens=v["tokens"], out_tokens=v["out"],
                n_out=v["n_out"], best=v["best"], new_window=v["new"], accept_len=v["accept"])


def _window_desc(v):
    return dict(logits_cur=v["cur"], logits_look=v["look"], out_tokens=v["out"], n_out=v["n_out"], best=v["best"], new_window=v["new"])


def _sample_desc(v):
    return dict(logits_cur=v["cur"], logits_cand=v["cand"], cand_tokens=v["tokens"], u_test=v["u_test"], u_final=v["u_final"],
                temperature=0.8, out_tokens=v["out"], n_out=v["n_out"])


def _table(x, first, pages):
    order = list(range(first, first + pages))
    x.host.shuffle(order)
    return torch.tensor(order, dtype=torch.int32, device="cuda")


def _prepare_loop(case, seed):
    host = random.Random(seed)
    prompts = [[0] + [host.randrange(1, wl.TOY_VOCAB) for _ in range(case["prompt"] - 1)] for _ in range(case["seqs"])]
    # (side by side the sequences run on until the slowest has its tokens)
    length = case["prompt"] + case["tokens"] * (1 if case["seqs"] == 1 else case["N"]) + 64
    if case["seqs"] == 1:
        model = lookahead.ToyAttentionLM(seed % 1000, max_len=length, page_size=case["page"] or None)
    else:
        model = lookahead.ToyBatchLM(seed % 1000, case["seqs"], max_len=length, page_size=case["page"])
    return dict(case=case, model=model, prompts=prompts, seed=seed)


def prepare(case, seed):
    if case["kind"] == "loop":
        return _prepare_loop(case, seed)
    x = _Inputs(seed)
    W, N, G, H, KV, d, L, V = (case[k] for k in ("W", "N", "G", "heads", "kv_heads", "head_dim", "layers", "V"))
    kind, cache, T = case["kind"], case.get("cache", "packed"), _rows(case)
    s = dict(case=case)
    if kind == "share":
        ids = lookahead.lp_share(W, N, G, case["parts"], case["part"])
        T = len(ids)
        s["ids"] = torch.tensor(ids, dtype=torch.int32, device="cuda")
    prefixes, page = _prefixes(case), case.get("page", 0)
    B = len(prefixes)
    q, out = x.normal(B, L, T, H, d), torch.empty((B, L, T, H, d), dtype=torch.bfloat16, device="cuda")
    if cache == "fp8":
        sk, sv = x.codes(B, L, T, KV, d), x.codes(B, L, T, KV, d)
        s["scales"] = torch.full((2, L, KV), 4.0 / 448.0, device="cuda") * (0.75 + 0.5 * x.uniform(2, L, KV))
    else:
        sk, sv = x.normal(B, L, T, KV, d), x.normal(B, L, T, KV, d)
    s.update(q=[list(t) for t in q], sk=[list(t) for t in sk], sv=[list(t) for t in sv], out=[list(t) for t in out], out_all=out)
    if cache == "rope":
        cos, sin = wl.rope_tables(prefixes[0] + W + N, d)
        s["cos"], s["sin"] = torch.from_numpy(cos).cuda(), torch.from_numpy(sin).cuda()
    if cache == "paged":
        need = [-(-(P + N) // page) for P in prefixes]
        first = [sum(need[:i]) for i in range(B)]
        kc, vc = (x.normal(L, sum(need), KV, page, d) for _ in range(2))
        s["tables"] = [_table(x, f, n) for f, n in zip(first, need)]
        s["kc"], s["vc"], s["kept"] = list(kc), list(vc), [kc, vc]
    else:
        def caches(P):
            if cache == "fp8":
                return x.codes(L, KV, P, d)
            rows = -(-(P + N) // 256) * 256 + 256 if cache == "inplace" else P   # in place: room to grow
            return x.normal(L, KV, rows, d)
        both = [(caches(P), caches(P)) for P in prefixes]
        s["kc"], s["vc"] = [list(k) for k, _ in both], [list(v) for _, v in both]
        s["kept"] = [t for pair in both for t in pair] if cache == "inplace" else []
        if kind != "batch":
            s["kc"], s["vc"] = s["kc"][0], s["vc"][0]
    if kind == "call":
        s["logits"] = x.normal(G, N - 1, V, dtype=torch.float32)
        s["tokens"] = s["logits"].argmax(-1).to(torch.int32)
        s["tokens"][::2, (N - 1) // 2] = 0                                       # every other candidate stops half way
        s["accept"], s["accepted"] = _ints(G), _ints(G, N - 1)
        return s
    if kind == "share":
        return s
    s["verify"] = [_plant(x, V, W, N, G) for _ in range(B)]
    s["results"] = dict(out=_ints(B, N), n_out=_ints(B, 1), best=_ints(B, 1), new=_ints(B, W), accept=_ints(B, G))
    for b, v in enumerate(s["verify"]):
        v.update({k: t[b] for k, t in s["results"].items()})
    if kind == "batch":
        s["steps"] = [[dict(q=s["q"][b][l], step_k=s["sk"][b][l], step_v=s["sv"][b][l], out=s["out"][b][l], P=P,
                            **({"block_table": s["tables"][b]} if cache == "paged" else
                               {"k_cache": s["kc"][b][l], "v_cache": s["vc"][b][l]}))
                       for b, P in enumerate(prefixes)] for l in range(L)]
        s["ends"] = [(_window_desc if case["sampling"] else _verify_desc)(v) for v in s["verify"]]
        s["samples"] = [_sample_desc(v) for v in s["verify"]]
    if cache in ("inplace", "paged"):
        s["appends"] = [dict(k_cache=s["kc"][l], v_cache=s["vc"][l], step_k=s["sk"][b][l], step_v=s["sv"][b][l],
                             best=s["verify"][b]["best"], n_out=s["verify"][b]["n_out"], P=P,
                             **({"block_table": s["tables"][b]} if cache == "paged" else {}))
                        for b, P in enumerate(prefixes) for l in range(L)]
    return s


# ---- one pass ----------------------------------------------------------------------------------

def _run_loop(s):
    case, model = s["case"], s["model"]
    if case["seqs"] == 1:
        model.length = 0                                     # a new generation on the model's cache
        dec = lookahead.LookaheadDecoder(model, s["prompts"][0], case["W"], case["N"], case["G"], seed=s["seed"],
                                         prompt_as_reference=True, temperature=case["temperature"] or None)
    else:
        model.lengths = [0] * case["seqs"]
        dec = lookahead.BatchedLookaheadDecoder(model, s["prompts"], case["W"], case["N"], case["G"],
                                                prompt_as_reference=True)
    return np.array(dec.generate(case["tokens"]), dtype=np.int64)


def _pick(v):
    """What a sampling program does between verification and append: read the tokens, find the
    candidate that starts with them."""
    n = int(v["n_out"].item())
    k, got = n - 1, v["out"][:n].tolist()
    v["best"].fill_(next((i for i, t in enumerate(v["toks"]) if t[:k] == got[:k]), -1) if k else -1)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "loop":
        return _run_loop(s)
    W, N, G, H, KV, d, L, V = (case[k] for k in ("W", "N", "G", "heads", "kv_heads", "head_dim", "layers", "V"))
    kc, vc = s["kc"], s["vc"]
    if kind == "batch":
        for l in range(L):
            if case["cache"] == "paged":
                binding.la_step_attention_batch_paged(s["steps"][l], kc[l], vc[l], W, N, G, H, KV, d)
            else:
                binding.la_step_attention_batch(s["steps"][l], W, N, G, H, KV, d)
        binding.la_verify_step_batch(s["ends"], W, N, 0 if case["sampling"] else G, V)
        if case["sampling"]:
            binding.la_verify_sample_batch(s["samples"], N, G, V)
        elif "appends" in s:
            binding.la_kv_commit_batch(s["appends"], W, N, G, KV, d)
        return [s["out_all"], s["kept"], s["results"]]
    P, q, sk, sv, out = case["P"], s["q"][0], s["sk"][0], s["sv"][0], s["out"][0]
    if kind == "share":
        for l in range(L):
            binding.la_step_attention_rows(q[l], kc[l], vc[l], sk[l], sv[l], s["ids"], P, W, N, G, H, KV, d, out[l])
        return s["out_all"]
    if kind == "call":
        binding.la_step_attention(q[0], kc[0], vc[0], sk[0], sv[0], P, W, N, G, H, KV, d, out[0])
        binding.la_verify(s["logits"], s["tokens"], G, N, V, s["accept"], s["accepted"])
        return [s["out_all"], s["accept"], s["accepted"]]
    cache = case["cache"]
    for l in range(L):
        if cache == "inplace":
            binding.la_step_attention_cap(q[l], kc[l], vc[l], sk[l], sv[l], P, W, N, G, H, KV, d, out[l])
        elif cache == "paged":
            binding.la_step_attention_paged(q[l], kc[l], vc[l], s["tables"][0], sk[l], sv[l], P, W, N, G, H, KV, d, out[l])
        elif cache == "rope":
            binding.la_step_attention_rope(q[l], kc[l], vc[l], sk[l], sv[l], s["cos"], s["sin"], P, W, N, G, H, KV, d, out[l],
                                           rotate_keys=True)
        else:
            binding.la_step_attention_fp8kv(q[l], kc[l], vc[l], sk[l], sv[l], s["scales"][0][l], s["scales"][1][l], P, W, N, G,
                                            H, KV, d, out[l])
    v = s["verify"][0]
    if case["sampling"]:
        binding.la_verify_step(v["cur"], v["look"], None, None, W, N, 0, V, v["out"], v["n_out"], v["best"], v["new"])
        binding.la_verify_sample(v["cur"], v["cand"], v["tokens"], v["u_test"], v["u_final"], 0.8, N, G, V, v["out"], v["n_out"])
        _pick(v)
    else:
        binding.la_verify_step(v["cur"], v["look"], v["cand"], v["tokens"], W, N, G, V, v["out"], v["n_out"], v["best"],
                               v["new"], v["accept"])
    if "appends" in s:
        binding.la_kv_commit_batch(s["appends"], W, N, G, KV, d)
    return [s["out_all"], s["kept"], s["results"]]
