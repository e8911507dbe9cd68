"""Lookups of present and absent segments in groups of every directory size (one entry, entries
shared by several lists, lists that share a bit), with exact and hashed segment keys: tau = 0 joins
of two sets, whose pairs are the equal strings (a host dictionary gives them)."""
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


# string length 4: keys are the packed symbols; 30: a hash.  256 symbols: packed up to 4 bytes
@pytest.mark.parametrize("length,symbols", [(4, 26), (30, 26), (3, 256), (12, 256)])
@pytest.mark.parametrize("lists", [1, 2, 3, 4, 5, 8, 9, 32, 33, 64, 65, 127, 129, 5000])
def test_group_sizes(length, symbols, lists):
    rng = np.random.default_rng(lists * 1000 + length)
    print("lists", lists, "length", length, "symbols", symbols, flush=True)
    base = 97 if symbols == 26 else 0
    words = set()
    while len(words) < lists:
        words.add((base + rng.integers(0, symbols, size=length)).astype(np.uint8).tobytes())
    words = sorted(words)
    # a second, empty-looking neighbourhood: one string of another length, so that groups without
    # lists lie between groups with some
    indexed = words + [words[0] + b"a" * 7]
    probes = [words[k] for k in rng.integers(0, lists, size=300)]
    for k in range(2000):           # absent ones: one symbol of a present one replaced
        w = bytearray(words[int(rng.integers(lists))])
        w[int(rng.integers(length))] = base + int(rng.integers(symbols))
        probes.append(bytes(w))
    got = P.pj_join(W.from_list(probes), W.from_list(indexed), 0)
    at = {w: k for k, w in enumerate(indexed)}
    exp = np.array([(q, at[w]) for q, w in enumerate(probes) if w in at], dtype=np.int32)
    assert np.array_equal(got, exp)
    assert P.pj_last_stats()["candidates"] == len(exp)
