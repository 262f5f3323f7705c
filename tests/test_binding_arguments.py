"""What the binding refuses before anything reaches the library: tensors of the wrong kind, place,
type, shape or layout raise, and name the argument."""
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
