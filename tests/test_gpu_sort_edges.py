"""The compaction of run heads at the edges of its tiles of 8,192 (from one tile, without look-back, to
several), through tau = 0 joins as the other sizes of sorts are tested, and an index of more than 2^30
entries, whose sorts take 64-bit status words.  Whole numbers: compared exactly."""
import numpy as np
import pytest

import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.load()
    yield


def _copies(words, pairs):
    """The distinct words, the first `pairs` of them twice, in random order: that many pairs."""
    rng = np.random.default_rng(pairs)
    order = rng.permutation(np.concatenate([np.arange(len(words)), np.arange(pairs)]))
    strings = [words[k] for k in order]
    first, exp = {}, []
    for k, s in enumerate(strings):
        if s in first:
            exp.append((first[s], k))
        else:
            first[s] = k
    return strings, np.array(sorted(exp), np.int32).reshape(-1, 2)


def _check(strings, exp):
    got = P.pj_self_join(W.from_list(strings), 0)
    assert P.pj_last_stats()["index_entries"] == len(strings)
    assert np.array_equal(got, exp)


@pytest.mark.parametrize("n", [8191, 8192, 8193, 16_383, 16_384, 16_385, 65 * 8192 + 1])
def test_index_entries(n):
    print("index entries", n, flush=True)
    _check(*_copies([b"%08d" % k for k in range(n - n // 3)], n // 3))


@pytest.mark.parametrize("pairs", [8191, 8193, 16_384, 16_385, 70_000])
def test_pairs(pairs):
    print("pairs", pairs, flush=True)
    _check(*_copies([b"%08d" % k for k in range(pairs + 5)], pairs))


def test_more_than_two_to_the_thirty():
    import torch
    n = (1 << 30) + 4097
    gen = torch.Generator(device="cuda").manual_seed(30)
    chars = torch.randint(0, 250, (n,), dtype=torch.uint8, device="cuda", generator=gen)
    rare = torch.unique(torch.cat([torch.randint(0, n, (1000,), device="cuda", generator=gen),
                                   torch.tensor([0, 4095, 4096, (1 << 30) - 1, 1 << 30, n - 1], device="cuda")]))
    chars[rare] = 255
    offs = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    print("index of", n, "strings of one byte", flush=True)
    index = P.pj_build_index((chars, offs), 0, 0)
    assert P.pj_last_stats()["index_entries"] == n
    for byte in (255, 7, 251):
        print("query", byte, flush=True)
        got = P.pj_query(index, W.from_list([bytes([byte])]), np.zeros(1, np.int32))
        exp = torch.nonzero(chars == byte)[:, 0].cpu().numpy()
        assert (got[:, 0] == 0).all() and np.array_equal(got[:, 1], exp)
    index.free()
