"""The decoding loop's host work in the extension module against its definitions in Python: the random
window levels, the draws of sampling, the pool's order, uploads."""
import random

import pytest
import torch

from paper_2402_02057_amd import binding, lookahead, workloads as wl


@pytest.mark.parametrize("seed", [0, 3, -7, 2**40 + 1, 2**70])
@pytest.mark.parametrize("count", [0, 1, 15, 61])
def test_generators_equal_their_definitions(seed, count):
    for step in (-4, -1, 0, 1, 1000):
        assert binding._native.window_random_tokens(seed, step, wl.TOY_VOCAB, count) == \
            [wl.window_random_token(seed, step, j) for j in range(count)]
        assert binding._native.uniform_draws(seed, step, 5, count) == \
            [float(wl.uniform_draw(seed, step, 5 + j)) for j in range(count)]


@pytest.mark.parametrize("vocab", [1, 0, -5, -2**63, 2**64 + 1, 2**70])
def test_random_tokens_of_no_vocabulary(vocab):
    with pytest.raises(ValueError):
        binding._native.window_random_tokens(1, 2, vocab, 3)
    assert binding._native.window_random_tokens(1, 2, 2, 3) == [1, 1, 1]


def test_pool_keeps_the_most_recent_last():
    rng, pool, want = random.Random(1), lookahead.NgramPool(), {}
    for _ in range(2000):
        gram = tuple(rng.randrange(4) for _ in range(4))
        pool.add(gram)
        bucket = want.setdefault(gram[0], [])
        if gram[1:] in bucket:
            bucket.remove(gram[1:])
        bucket.append(gram[1:])
    for first in range(5):
        for limit in (0, 1, 7, 1000):
            assert pool.lookup(first, limit) == (want.get(first, [])[-limit:] if limit else [])


def test_what_is_not_in_range_is_not_uploaded():
    for lists in ([[0, 10]], [[-1]], [[2**70]], [[True]], [[1.0]], [(1,)], ([1],), [1], None, [[1], None]):
        assert binding._native.upload_in_range(lists, 10) is None
    assert binding._native.upload_in_range([[2**31]], 2**40) is None


def test_lookup_reads_no_more_than_it_returns():
    class Bucket(dict):
        read = 0

        def __iter__(self):
            raise AssertionError("the whole bucket is read")

        def __reversed__(self):
            for key in dict.__reversed__(self):
                self.read += 1
                yield key
    pool = lookahead.NgramPool()
    pool._tails[3] = bucket = Bucket()
    for i in range(1000):
        pool.add((3, i, i + 1))
    assert pool.lookup(3, 4) == [(i, i + 1) for i in range(996, 1000)] and bucket.read == 4


@pytest.mark.gpu
def test_uploads_in_range():
    assert binding._native.upload_in_range([[0, 5], [], [9]], 10).tolist() == [0, 5, 9]
    assert binding._native.upload_in_range([], 10).numel() == 0 and binding._native.upload_in_range([[1]], 2).dtype == torch.int32


@pytest.mark.gpu
def test_uploads():
    sent = []
    for i in range(200):                       # none is waited for: each keeps its numbers until it has run
        lists = [[i * 1000 + j for j in range(i % 7)], [], [-1, 2**31 - 1, -2**31]]
        sent.append((sum(lists, []), binding._native.upload(lists, False)))
    for want, got in sent:
        assert got.dtype == torch.int32 and got.is_cuda and got.tolist() == want
    assert binding._native.upload([[0.5, 1], [2.0**-24]], True).tolist() == [0.5, 1.0, 2.0**-24]
    assert binding._native.upload([], False).numel() == 0
    for bad, error in ((((1,),), TypeError), ([(1,)], TypeError), ([["a"]], TypeError), ([[2**31]], ValueError)):
        with pytest.raises(error):
            binding._native.upload(bad, False)


class Clears:
    """An int whose conversion changes the lists that it is in."""

    def __init__(self, lists, do):
        self.lists, self.do = lists, do

    def __index__(self):
        self.do(self.lists)
        return 7


@pytest.mark.gpu
@pytest.mark.parametrize("do,want", [(lambda l: l.clear(), [1, 7, 2, 3]), (lambda l: l[0].clear(), [1, 7, 4, 5]),
                                     (lambda l: l.__setitem__(1, [9]), [1, 7, 2, 3, 9]), (lambda l: l.pop(), [1, 7, 2, 3])])
def test_uploads_of_lists_that_change(do, want):
    lists = []
    lists += [[1, Clears(lists, do), 2, 3], [4, 5]]
    assert binding._native.upload(lists, False).tolist() == want
    lists[:] = [[1, Clears(lists, lambda l: l.__setitem__(1, None)), 2, 3], [4, 5]]
    with pytest.raises(TypeError):
        binding._native.upload(lists, False)
