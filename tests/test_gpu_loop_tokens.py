"""GPU: the tokens that the toy models' forward pass and the decoding loop take: every form that torch.tensor takes."""
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
