"""The device-wide sort, scan and compaction at the edges of their tiles, through tau = 0
self-joins: every string is one index entry, so the set's size is the sort's, and the pairs are
those of equal strings (ED = 0), found here by sorting the strings on the host.  Whole numbers:
the results are compared exactly."""
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


def _equal_pairs(strings):
    order = sorted(range(len(strings)), key=lambda k: (strings[k], k))
    pairs, group = [], [order[0]]
    for k in order[1:]:
        if strings[k] == strings[group[0]]:
            pairs.extend((g, k) for g in group)
            group.append(k)
        else:
            group = [k]
    return np.array(sorted(pairs), dtype=np.int32).reshape(-1, 2)


def _check(strings):
    got = P.pj_self_join(W.from_list(strings), 0)
    st = P.pj_last_stats()
    exp = _equal_pairs(strings)
    assert st["index_entries"] == len(strings)
    assert np.array_equal(got, exp)


# a tile holds 1024 keys below 2^18 and 4096 from there on; a scan or compaction tile 2048
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4097,
                               66_000, (1 << 18) - 1, 1 << 18, (1 << 18) + 4097, 401_409])
def test_index_sizes(n):
    rng = np.random.default_rng(n)
    print("index entries", n, flush=True)
    lens = rng.integers(1, 40, size=max(n * 4 // 5, 1))
    chars = rng.integers(97, 123, size=int(lens.sum())).astype(np.uint8).tobytes()
    at = np.concatenate([[0], np.cumsum(lens)])
    words = [chars[at[k]:at[k + 1]] for k in range(len(lens))]
    # (words of one letter repeat by the thousand in the larger sets: keep those of 4 or more)
    words = [w for w in words if len(w) >= 4] or words[:1]
    _check([words[k] for k in rng.integers(0, len(words), size=n)])


# accepted candidates (= pairs at tau = 0): one block up to 4096, the radix sort beyond
@pytest.mark.parametrize("pairs", [1, 63, 64, 65, 128, 129, 1023, 1025, 2048, 4095, 4096, 4097, 8192])
def test_pair_counts(pairs):
    rng = np.random.default_rng(pairs)
    print("accepted candidates", pairs, flush=True)
    words = [b"%08d" % k for k in rng.permutation(pairs + 100)]
    _check([words[k] for k in rng.permutation(np.concatenate([np.arange(len(words)),
                                                              np.arange(pairs)]))])


# one list with every string: one run across many tiles, every digit of every key the same
def test_one_list():
    print("one list", flush=True)
    _check([b"same"] * 3000)
