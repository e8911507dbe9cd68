"""pj_query on both sides of its small-batch route (one upload, sizes kept on the device): numbers of
queries around its limit, results that need the second read-back, and results or candidates beyond
its buffers, which the general path takes.  Pairs and counts equal pj_join's of the same sets, whose
pairs the oracle's tests pin; a brute-force join checks the pairs again."""
import numpy as np
import pytest

import oracle as O
import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.load()
    yield


def _check(index_strings, queries, tau):
    S, Q = W.from_list(index_strings), W.from_list(queries)
    joined = P.pj_join(Q, S, tau)
    sj = P.pj_last_stats()
    idx = P.pj_build_index(S, 0, tau)
    for _ in range(2):                     # a second call on the same buffers
        got = P.pj_query(idx, Q, np.full(Q.n, tau, np.int32))
        st = P.pj_last_stats()
        assert np.array_equal(got, joined)
        for k in ("selected", "hits", "candidates", "cells", "accepted", "side_pairs", "pairs"):
            assert st[k] == sj[k], k
    idx.free()
    return joined, S, Q


@pytest.mark.parametrize("n", [1, 2, 63, 65, 511, 512, 513])
def test_numbers_of_queries(n):
    rng = np.random.default_rng(n)
    print("queries", n, flush=True)
    base = W.cfg2(3000, seed=5).as_list()
    ed = W._Editor(rng, W.ALPHA27, W.english27_probs())
    queries = [ed.edit(base[int(rng.integers(len(base)))], int(rng.integers(0, 4))) for _ in range(n)]
    joined, S, Q = _check(base, queries, 2)
    assert np.array_equal(joined, O.join_bf(Q, S, 2))


# 1024: the pairs read back at once; 8192: accepted candidates the batch can sort (equal strings are
# accepted once per slot, 3 times at tau = 2)
@pytest.mark.parametrize("equal", [1, 340, 1023, 1024, 1025, 2730, 2731, 9000])
def test_result_sizes(equal):
    print("equal strings", equal, flush=True)
    strings = [b"the quick brown fox"] * equal + [b"jumps over the lazy dog"] * 5
    joined, _, _ = _check(strings, [b"the quick brown fox", b"jumps over the hazy dog", b"nothing"], 2)
    assert len(joined) == equal + 5


def test_candidates_beyond_the_buffers():
    # one-letter segments: every string of the list is a candidate in every slot
    rng = np.random.default_rng(3)
    strings = [bytes(rng.integers(97, 99, size=6).astype(np.uint8)) for _ in range(4000)]
    queries = [bytes(rng.integers(97, 99, size=6).astype(np.uint8)) for _ in range(200)]
    print("candidates", flush=True)
    _check(strings, queries, 4)


def test_short_strings_and_empty_results():
    print("short", flush=True)
    _check([b"", b"a", b"ab", b"abc", b"zzzzzzzz"], [b"", b"b", b"qqqqqqqqqqqq"], 2)
