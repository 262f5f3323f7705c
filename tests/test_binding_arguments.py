"""What the binding refuses before anything reaches the library: tensors of the wrong kind, place,
type, shape or layout raise, and name the argument."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2402_02057_amd import binding

H, KV, D, P, W, N, G = 4, 2, 64, 3, 2, 3, 1
T = 1 + (W + G) * (N - 1)
SHAPES = {"q": (T, H, D), "k_cache": (KV, P, D), "v_cache": (KV, P, D), "step_k": (T, KV, D), "step_v": (T, KV, D),
          "out": (T, H, D)}


def tensors(device):
    return {k: torch.zeros(s, dtype=torch.bfloat16, device=device) for k, s in SHAPES.items()}


def step(x, **sizes):
    s = dict(dict(P=P, W=W, N=N, G=G, heads=H, kv_heads=KV, head_dim=D), **sizes)
    return binding.la_step_attention(x["q"], x["k_cache"], x["v_cache"], x["step_k"], x["step_v"], out=x["out"], **s)


BF, F, I, U = torch.bfloat16, torch.float32, torch.int32, torch.uint8
V, CAP, PAGE, POS = 50, 16, 64, 32
STEP = {"P": P, "W": W, "N": N, "G": G, "heads": H, "kv_heads": KV, "head_dim": D}
CACHE = {"k_cache": ((KV, P, D), BF), "v_cache": ((KV, P, D), BF)}
PAGES = {"k_pages": ((2, KV, PAGE, D), BF), "v_pages": ((2, KV, PAGE, D), BF)}
ROOM = {"k_cache": ((KV, CAP, D), BF), "v_cache": ((KV, CAP, D), BF)}
ROWS = {"q": ((T, H, D), BF), "step_k": ((T, KV, D), BF), "step_v": ((T, KV, D), BF), "out": ((T, H, D), BF)}
KEYS = {"step_k": ((T, KV, D), BF), "step_v": ((T, KV, D), BF)}
TABLES = {"cos": ((POS, D // 2), F), "sin": ((POS, D // 2), F)}
ENDED = {"best": ((1,), I), "n_out": ((1,), I)}
GREEDY = {"logits_cur": ((V,), F), "logits_look": ((W, V), F), "logits_cand": ((G, N - 1, V), F), "cand_tokens": ((G, N - 1), I),
          "out_tokens": ((N,), I), "n_out": ((1,), I), "best": ((1,), I), "new_window": ((W,), I), "accept_len": ((G,), I)}
SAMPLED = {"logits_cur": ((V,), F), "logits_cand": ((G, N - 1, V), F), "cand_tokens": ((G, N - 1), I), "u_test": ((N - 1, G), F),
           "u_final": ((1,), F), "out_tokens": ((N,), I), "n_out": ((1,), I)}
# every entry point: its tensors (of a descriptor, in a batch), the sizes it takes, and a batch's own tensors
ENTRIES = {
    "la_step_attention": (dict(ROWS, **CACHE), STEP),
    "la_step_attention_noalloc": (dict(ROWS, **CACHE), STEP),
    "la_step_attention_fp8kv": (dict(ROWS, **{k: (v[0], U) for k, v in dict(CACHE, **KEYS).items()}, k_scale=((KV,), F), v_scale=((KV,), F)), STEP),
    "la_step_attention_cap": (dict(ROWS, **ROOM), STEP),
    "la_step_rope": (dict({k: ROWS[k] for k in ("q", "step_k")}, **TABLES), STEP),
    "la_step_attention_rope": (dict(ROWS, **CACHE, **TABLES), STEP),
    "la_step_attention_rows": (dict(ROWS, **CACHE, row_ids=((T,), I)), STEP),
    "la_step_attention_paged": (dict(ROWS, **PAGES, block_table=((1,), I)), STEP),
    "la_kv_commit": (dict(KEYS, **ROOM, **ENDED), {k: v for k, v in STEP.items() if k != "heads"}),
    "la_kv_commit_rope": (dict(KEYS, **ROOM, **TABLES, **ENDED), {k: v for k, v in STEP.items() if k != "heads"}),
    "la_kv_commit_paged": (dict(KEYS, **PAGES, block_table=((1,), I), **ENDED), {k: v for k, v in STEP.items() if k != "heads"}),
    "la_verify": ({"logits": ((G, N - 1, V), F), "cand_tokens": ((G, N - 1), I), "accept_len": ((G,), I), "accepted": ((G, N - 1), I)},
                  dict(G=G, N=N, V=V)),
    "la_verify_step": (GREEDY, dict(W=W, N=N, G=G, V=V)),
    "la_verify_sample": (SAMPLED, dict(temperature=0.8, N=N, G=G, V=V)),
    "la_step_attention_batch": (dict(ROWS, **CACHE), {k: v for k, v in STEP.items() if k != "P"}, {}),
    "la_step_attention_batch_paged": (dict(ROWS, block_table=((1,), I)), {k: v for k, v in STEP.items() if k != "P"}, PAGES),
    "la_kv_commit_batch": (dict(KEYS, **ROOM, **ENDED), dict(W=W, N=N, G=G, kv_heads=KV, head_dim=D), {}),
    "la_verify_step_batch": (GREEDY, dict(W=W, N=N, G=G, V=V), {}),
    "la_verify_sample_batch": (SAMPLED, dict(N=N, G=G, V=V), {}),
}


def call(entry, change=None, device="cuda"):
    """The entry point with all its tensors as they should be, but for the one named `change`."""
    made, sizes, *batch = ENTRIES[entry]

    def make(tensors):
        x = {k: torch.zeros(shape, dtype=dtype, device=device) for k, (shape, dtype) in tensors.items()}
        return {k: v.to({BF: F, F: torch.float64, I: torch.int64, U: torch.int8}[v.dtype]) if k == change else v for k, v in x.items()}
    f = getattr(binding, entry)
    if not batch:
        return f(**make(made), **sizes)
    descs = [dict(make(made), P=P, temperature=0.8) for _ in range(2)]
    return f(descs, **make(batch[0]), **sizes)


@pytest.mark.parametrize("entry", sorted(ENTRIES))
def test_every_entry_point_refuses_host_tensors(entry):
    with pytest.raises(ValueError, match="must live on the GPU"):
        call(entry, device="cpu")


@pytest.mark.gpu
@pytest.mark.parametrize("entry", sorted(ENTRIES))
def test_every_entry_point_checks_every_tensor(entry):
    call(entry)
    torch.cuda.synchronize()
    for name in list(ENTRIES[entry][0]) + list(ENTRIES[entry][2] if len(ENTRIES[entry]) > 2 else []):
        with pytest.raises(ValueError, match="^%s must be torch" % name):
            call(entry, change=name)


@pytest.mark.parametrize("name, value, error, text", [
    ("q", None, ValueError, "q is None"),
    ("q", [1.0], TypeError, "q must be a torch.Tensor"),
    ("q", "host", ValueError, "q must live on the GPU"),
])
def test_refused_without_a_gpu(name, value, error, text):
    x = tensors("cpu")
    if value != "host":
        x[name] = value
    with pytest.raises(error, match=text):
        step(x)
    with pytest.raises(KeyError, match="P"):
        binding.la_step_attention_batch([{}], W, N, G, H, KV, D)
    with pytest.raises(TypeError):
        step(tensors("cpu"), W="2")


@pytest.mark.parametrize("name", ["P", "W", "N", "G", "heads", "kv_heads", "head_dim"])
@pytest.mark.parametrize("by", [1 << 32, -(1 << 32), 1 << 31, 1 << 64, -(1 << 80)])
def test_sizes_that_do_not_fit_are_refused(name, by):
    """Before the tensors are looked at, which live on the host here: the rest of 2^32 fits them."""
    right = dict(P=P, W=W, N=N, G=G, heads=H, kv_heads=KV, head_dim=D)
    with pytest.raises(ValueError, match="%d does not fit 32 bits" % (right[name] + by)):
        step(tensors("cpu"), **{name: right[name] + by})
    if name == "P":
        with pytest.raises(ValueError, match="does not fit 32 bits"):
            binding.la_step_attention_batch([dict(tensors("cpu"), P=P + by)], W, N, G, H, KV, D)
        with pytest.raises(ValueError, match="does not fit 32 bits"):
            binding.la_step_attention_batch([dict(tensors("cpu"), P=str(P + by))], W, N, G, H, KV, D)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_refused_on_the_gpu(name):
    good = tensors("cuda")
    assert step(good) is good["out"]
    with pytest.raises(ValueError, match=r"%s must have shape \(%s\), got \(%d, " % (name, ", ".join(map(str, SHAPES[name])), SHAPES[name][0] + 1)):
        step(dict(good, **{name: torch.zeros((SHAPES[name][0] + 1,) + SHAPES[name][1:], dtype=torch.bfloat16, device="cuda")}))
    with pytest.raises(ValueError, match="%s must be torch.bfloat16, got torch.float32" % name):
        step(dict(good, **{name: good[name].float()}))
    with pytest.raises(ValueError, match="%s must be contiguous" % name):
        step(dict(good, **{name: torch.zeros(SHAPES[name] + (2,), dtype=torch.bfloat16, device="cuda")[..., 0]}))
    with pytest.raises(ValueError, match="%s must live on the GPU" % name):
        step(dict(good, **{name: good[name].cpu()}))


class Made:
    """A descriptor that makes its values when it is asked for them: nobody else holds them."""

    def __init__(self, values):
        self.values = values

    def __getitem__(self, key):
        v = self.values[key]
        return v.view(v.shape) if isinstance(v, torch.Tensor) else int(str(v)) if isinstance(v, int) else v


MADE_ON_ACCESS = """
import torch
from paper_2402_02057_amd import binding

class Made:
    def __getitem__(self, key):
        return int("123456789") if key == "P" else torch.zeros(1, 2, 64, 64)

for call in (lambda x: binding.la_step_attention_batch(x, 2, 3, 1, 4, 2, 64),
             lambda x: binding.la_step_attention_batch_paged(x, torch.zeros(1, 2, 64, 64), torch.zeros(1, 2, 64, 64), 2, 3, 1, 4, 2, 64),
             lambda x: binding.la_kv_commit_batch(x, 2, 3, 1, 2, 64),
             lambda x: binding.la_verify_step_batch(x, 2, 3, 1, 50),
             lambda x: binding.la_verify_sample_batch(x, 3, 1, 50)):
    try:
        call([Made()])
        raise SystemExit("accepted")
    except ValueError as e:
        print(e)
"""


def test_values_made_on_access_are_held():
    """Under Python's debugging allocator, which overwrites what is freed."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", MADE_ON_ACCESS], cwd=root, env=dict(os.environ, PYTHONMALLOC="debug"),
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert r.stdout.count("GPU") >= 3 and "block_table must hold at least" in r.stdout, r.stdout


class Answering(dict):
    """A dict that answers for itself: missing keys, and another value than the one it stores."""

    def __missing__(self, key):
        raise RuntimeError("asked for " + key)

    def __getitem__(self, key):
        return None if key == "q" else super().__getitem__(key)


def test_dict_subclasses_answer_for_themselves():
    with pytest.raises(RuntimeError, match="asked for P"):
        binding.la_step_attention_batch([Answering()], W, N, G, H, KV, D)
    with pytest.raises(ValueError, match="q is None"):
        binding.la_step_attention_batch([Answering(tensors("cpu"), P=P)], W, N, G, H, KV, D)
    # an optional key is asked for with get(), which does not run __missing__
    with pytest.raises(ValueError, match="k_cache must live on the GPU"):
        binding.la_kv_commit_batch([Answering(tensors("cpu"), P=P)], W, N, G, KV, D)


@pytest.mark.gpu
@pytest.mark.parametrize("temperature", ["0.5", 0.5, torch.tensor(0.5), b"0.5"])
def test_temperature_is_anything_float_takes(temperature):
    V = 50
    logits = torch.linspace(0.0, 3.0, V, device="cuda")
    u = torch.full((1,), 0.25, device="cuda")
    outs = []
    for t in (temperature, 0.5):
        out, n_out = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in (N, 1))
        binding.la_verify_sample(logits, None, None, None, u, t, N, 0, V, out, n_out)
        batched, n_batched = torch.zeros_like(out), torch.zeros_like(n_out)
        binding.la_verify_sample_batch([dict(logits_cur=logits, u_final=u, temperature=t, out_tokens=batched, n_out=n_batched)], N, 0, V)
        outs += [out, batched]
        assert int(n_out) == int(n_batched) == 1
    assert all(torch.equal(o, outs[0]) for o in outs)
    with pytest.raises(ValueError, match="could not convert"):
        binding.la_verify_sample(logits, None, None, None, u, "warm", N, 0, V, out, n_out)


@pytest.mark.gpu
def test_descriptors_that_make_their_values_give_what_dicts_give():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    seqs = [dict({k: torch.randn(s, device="cuda", generator=gen).bfloat16() for k, s in SHAPES.items()}, P=P) for _ in range(3)]
    binding.la_step_attention_batch([Made(x) for x in seqs], W, N, G, H, KV, D)
    made = [x["out"].clone() for x in seqs]
    binding.la_step_attention_batch(seqs, W, N, G, H, KV, D)
    torch.cuda.synchronize()
    assert all(torch.equal(x["out"], m) for x, m in zip(seqs, made))


@pytest.mark.gpu
def test_streams_are_none_a_stream_or_a_handle():
    x = tensors("cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    class Handle:
        def __int__(self):
            return side.cuda_stream

    outs = []
    for stream in (None, side, side.cuda_stream, Handle(), 0, torch.cuda.ExternalStream(side.cuda_stream)):
        out = torch.full_like(x["out"], float("nan"))
        side.wait_stream(torch.cuda.current_stream())
        binding.la_step_attention(*(x[k] for k in ("q", "k_cache", "v_cache", "step_k", "step_v")), P, W, N, G, H, KV, D, out, stream)
        torch.cuda.synchronize()
        outs.append(out)
    assert all(torch.equal(o, outs[0]) and bool(torch.isfinite(o).all()) for o in outs)
    with pytest.raises(TypeError):
        binding.la_step_attention(*(x[k] for k in ("q", "k_cache", "v_cache", "step_k", "step_v")), P, W, N, G, H, KV, D, out, object())


@pytest.mark.gpu
def test_tuples_do_as_well_as_lists():
    x = dict(tensors("cuda"), P=P)
    for seqs in ([x, x], (x, x)):
        x["out"].fill_(float("nan"))
        binding.la_step_attention_batch(seqs, W, N, G, H, KV, D)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(x["out"]).all())


@pytest.mark.gpu
def test_a_list_that_grows_during_the_call_is_taken_as_it_was():
    class Growing(Made):
        def __getitem__(self, key):
            seqs.extend([self] * 64)
            return super().__getitem__(key)

    x = dict(tensors("cuda"), P=P)
    seqs = [Growing(x), Growing(dict(x, out=torch.full_like(x["out"], float("nan"))))]
    last = seqs[-1]
    binding.la_step_attention_batch(seqs, W, N, G, H, KV, D)
    torch.cuda.synchronize()
    assert len(seqs) > 64 and bool(torch.isfinite(last.values["out"]).all())
