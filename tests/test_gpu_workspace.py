"""What the attention calls take of device memory, and what a batch does where the pipelined kernel's partial
results have no room."""
import pytest
import torch

from paper_2402_02057_amd import binding

pytestmark = pytest.mark.gpu
MB = 1 << 20


def make_steps(prefixes, W, N, G, H, KV, d, seed=1):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    T = 1 + (W + G) * (N - 1)

    def rb(*shape):
        return torch.randn(shape, device="cuda", generator=gen).bfloat16()
    return [dict(q=rb(T, H, d), k_cache=rb(KV, P, d), v_cache=rb(KV, P, d), step_k=rb(T, KV, d), step_v=rb(T, KV, d), P=P,
                 out=torch.empty((T, H, d), dtype=torch.bfloat16, device="cuda")) for P in prefixes]


def run(steps, shape):
    W, N, G, H, KV, d = shape
    if len(steps) == 1:
        s = steps[0]
        binding.la_step_attention(s["q"], s["k_cache"], s["v_cache"], s["step_k"], s["step_v"], s["P"], *shape, s["out"])
    else:
        binding.la_step_attention_batch(steps, *shape)
    torch.cuda.synchronize()


@pytest.fixture
def fresh_set():
    """A workspace set that nobody has used since the library's blocks were last given back."""
    torch.cuda.synchronize()
    binding.la_shutdown()
    binding.la_select_workspace(12)
    yield
    binding.la_select_workspace(0)


@pytest.mark.parametrize("prefixes,shape,at_most", [
    ([1024], (15, 5, 15, 32, 32, 128), 33),                      # one step, cut
    ([3000, 900, 800], (3, 3, 3, 4, 4, 128), 33),                # one tile per KV head: no pipelined kernel
    ([3000, 900, 800], (15, 5, 15, 32, 8, 64), 33),              # nor for head_dim 64
    ([8000, 8000], (15, 5, 15, 32, 8, 128), 59),                   # pipelined, cut: 58 MB at once
], ids=["step", "few-rows", "head-dim-64", "pipelined"])
def test_device_memory_of_a_set(fresh_set, prefixes, shape, at_most):
    print("case", dict(prefixes=prefixes, shape=shape), flush=True)
    if len(prefixes) == 1:
        assert binding.la_step_attention_workspace_bytes(prefixes[0], *shape) > 0
    steps = make_steps(prefixes, *shape)
    binding.la_select_workspace(11)
    run(steps, shape)                       # (whatever the first launch of a kernel allocates)
    binding.la_select_workspace(12)
    before = torch.cuda.mem_get_info()[0]
    run(steps, shape)
    taken = before - torch.cuda.mem_get_info()[0]
    assert 0 < taken <= (at_most + 2) * MB, taken / MB       # (two blocks, each rounded up to at most a megabyte)


def test_a_batch_is_captured_after_a_step_alone(fresh_set, override):
    """The step's workspace holds the partial results of any batch of the staged kernel but not those of the pipelined
    one, and cannot grow inside the capture: the batch is recorded with the staged kernel, whose bits it has."""
    shape, prefixes = (15, 5, 15, 32, 8, 128), [8000, 8000]   # (pipelined and cut: test_launch_plan.py)
    steps = make_steps(prefixes, *shape)
    binding.la_select_workspace(11)
    run(steps, shape)                       # (kernels loaded ahead of the capture)
    pipelined = [s["out"].clone() for s in steps]
    override("batch_plan", "2")
    run(steps, shape)
    staged = [s["out"].clone() for s in steps]
    override("batch_plan", None)
    assert not all(torch.equal(a, b) for a, b in zip(pipelined, staged))
    binding.la_select_workspace(12)
    alone = (15, 5, 15, 32, 32, 128)
    assert binding.la_step_attention_workspace_bytes(1024, *alone) > 0
    run(make_steps([1024], *alone), alone)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.la_step_attention_batch(steps, *shape)
    for _ in range(3):
        for s in steps:
            s["out"].fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(s["out"], w) for s, w in zip(steps, staged))
        run(steps, shape)                   # eager again, now with the larger block
        assert all(torch.equal(s["out"], w) for s, w in zip(steps, pipelined))


def test_a_batch_cannot_be_captured_with_nothing_reserved(fresh_set):
    """It is refused, as ever, and not recorded as nothing."""
    shape = (15, 5, 15, 32, 8, 128)
    steps = make_steps([8000, 8000], *shape)
    binding.la_select_workspace(11)
    run(steps, shape)
    binding.la_select_workspace(12)
    x = torch.zeros(8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        with pytest.raises(binding.LaError):
            binding.la_step_attention_batch(steps, *shape)
    graph.replay()
    torch.cuda.synchronize()
    assert x.tolist() == [1.0] * 8
