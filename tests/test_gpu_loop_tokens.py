"""GPU: the tokens that the toy models' forward pass and the decoding loop take: every form that torch.tensor takes,
and a model of the caller's own that changes them, or runs on a stream of its own."""
import warnings

import numpy as np
import pytest
import torch

from paper_2402_02057_amd import lookahead, workloads as wl

pytestmark = pytest.mark.gpu
W, N, G = 5, 4, 3
T = 1 + (W + G) * (N - 1)


def tokens_of(seed):
    return [wl.window_random_token(seed, 1, j) for j in range(T)]


def single(page_size=None):
    model = lookahead.ToyAttentionLM(1, max_len=256, page_size=page_size)
    model.append([0, 5, 9, 4])
    return model


def batched():
    model = lookahead.ToyBatchLM(1, 2, max_len=256)
    for i in range(2):
        model.append(i, [0, 5, 9 + i])
    return model


FORMS = {"tuple": tuple, "numpy ints": lambda t: [np.int64(x) for x in t], "array": np.array,
         "floats": lambda t: [float(x) for x in t], "tensor": torch.tensor, "gpu tensor": lambda t: torch.tensor(t, device="cuda")}


@pytest.mark.parametrize("page_size", [None, 64])
@pytest.mark.parametrize("form", FORMS)
def test_forward_step_takes_any_form_of_tokens(form, page_size):
    model, tokens = single(page_size), tokens_of(3)
    want = model.forward_step(tokens, W, N, G)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")           # (torch.tensor of a tensor)
        assert torch.equal(model.forward_step(FORMS[form](tokens), W, N, G), want)
    assert want.shape == (T, wl.TOY_VOCAB)


@pytest.mark.parametrize("form", FORMS)
def test_batched_forward_step_takes_any_form_of_tokens(form):
    model, tokens = batched(), [tokens_of(3), tokens_of(4)]
    want = model.forward_step(tokens, W, N, G)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        forms = [[FORMS[form](t) for t in tokens]] if form != "gpu tensor" and form != "tensor" else []
        if form in ("array", "tensor", "gpu tensor"):
            forms.append(FORMS[form](tokens))
        for f in forms:
            assert all(torch.equal(a, b) for a, b in zip(model.forward_step(f, W, N, G), want))


def test_negative_tokens_count_from_the_end():
    tokens = tokens_of(3)
    tokens[2] = wl.TOY_VOCAB - 1
    turned = [t - wl.TOY_VOCAB if i % 3 == 2 else t for i, t in enumerate(tokens)]
    model = single()
    want = model.forward_step(tokens, W, N, G)
    for form in (turned, tuple(turned), np.array(turned), torch.tensor(turned, device="cuda")):
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            assert torch.equal(model.forward_step(form, W, N, G), want)
    model, two = batched(), [tokens, tokens_of(4)]
    for a, b in zip(model.forward_step([turned, two[1]], W, N, G), model.forward_step(two, W, N, G)):
        assert torch.equal(a, b)
    for wrong in (wl.TOY_VOCAB, -wl.TOY_VOCAB - 1, 2**40):
        with pytest.raises(IndexError):
            single().forward_step(tokens[:-1] + [wrong], W, N, G)
        with pytest.raises(IndexError):
            model.forward_step([tokens, tokens[:-1] + [wrong]], W, N, G)


def test_a_loop_with_negative_random_tokens():
    """(they stand for others of the vocabulary to the model, and are no candidates' tokens to the verification)"""
    runs = []
    for turn in (0, wl.TOY_VOCAB):
        runs.append(loop(lookahead.ToyAttentionLM(0), random_token=lambda *a: wl.window_random_token(*a) - turn))
    assert runs[0] == runs[1]


def loop(model, n_tokens=60, **more):
    """The tokens of a run; every step of the current stream starts behind some work."""
    dec, out = lookahead.LookaheadDecoder(model, [0, 5, 9, 5], W, N, G, **more), []
    torch.cuda.synchronize()
    while len(out) < n_tokens:
        torch.cuda._sleep(500000)
        out += dec.step()[0]
    return out[:n_tokens]


class Changes(lookahead.ToyAttentionLM):
    """Replaces a token of the window before the model runs."""

    def forward_step(self, tokens, W, N, G):
        tokens[1] = 1 + tokens[1] % (wl.TOY_VOCAB - 1)
        got = super().forward_step(tokens, W, N, G)
        assert torch.equal(got, super().forward_step([int(t) for t in tokens], W, N, G))
        return got


class ChangesBatch(lookahead.ToyBatchLM):
    def forward_step(self, tokens, W, N, G):
        tokens[1][1] = 1 + tokens[1][1] % (wl.TOY_VOCAB - 1)
        got = super().forward_step(tokens, W, N, G)
        assert all(torch.equal(a, b) for a, b in zip(got, super().forward_step([list(t) for t in tokens], W, N, G)))
        return got


def test_a_model_may_change_its_tokens():
    dec = lookahead.LookaheadDecoder(Changes(0), [0, 5, 9, 5], W, N, G)
    dec.generate(30)
    prompts = [[0, 5, 9], [0, 6, 9]]
    lookahead.BatchedLookaheadDecoder(ChangesBatch(0, 2, max_len=1024), prompts, W, N, G).generate(30)


@pytest.mark.parametrize("kind", [float, np.int64, np.float64])
def test_random_tokens_of_any_kind(kind):
    want = loop(lookahead.ToyAttentionLM(0))
    assert loop(lookahead.ToyAttentionLM(0), random_token=lambda *a: kind(wl.window_random_token(*a))) == want


class OnAStreamOfItsOwn(lookahead.ToyAttentionLM):
    """Its work waits for nothing of the caller's stream: the caller has read the last step's result."""

    def __init__(self, seed):
        super().__init__(seed)
        self.stream = torch.cuda.Stream()

    def forward_step(self, tokens, W, N, G):
        with torch.cuda.stream(self.stream):
            logits = super().forward_step(tokens, W, N, G)
        torch.cuda.current_stream().wait_stream(self.stream)
        return logits


def test_a_model_on_a_stream_of_its_own():
    assert loop(OnAStreamOfItsOwn(0)) == loop(lookahead.ToyAttentionLM(0))
