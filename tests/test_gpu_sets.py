"""How a set of strings is laid out on the device: the sort by length (one pass below 256 bytes, two
from there on) at the edges of its tiles, slots filled sixteen bytes at a time from any address, a
last string that ends with the bytes, empty strings and all byte values.  Pairs at tau = 1 and
candidates equal the oracle's."""
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


def _strings(rng, n, longest, values):
    """n strings of up to longest bytes, half of them one substitution away from another."""
    lens = rng.integers(0, longest + 1, size=n)
    lens[rng.integers(0, n)] = longest
    out = []
    for k, ln in enumerate(lens):
        if k % 2 and len(out[-1]):
            s = bytearray(out[-1])
            s[rng.integers(0, len(s))] = int(rng.integers(0, values))
            out.append(bytes(s))
        else:
            out.append(rng.integers(0, values, size=int(ln)).astype(np.uint8).tobytes())
    out.append(b"z" * longest)
    return out


# n: a sort tile holds 1024 ids; longest: a chunk is 16 bytes, one pass sorts lengths below 256;
# at: the bytes' address modulo 16
@pytest.mark.parametrize("at", [0, 1, 7, 15])
@pytest.mark.parametrize("n,longest", [(1, 0), (1, 16), (2, 15), (63, 17), (1023, 33), (1024, 64),
                                       (1025, 254), (900, 255), (900, 256), (2049, 40),
                                       (300, 1025), (60, 2047)])
def test_set_layout(n, longest, at):
    import torch
    rng = np.random.default_rng(1000 * n + longest + at)
    print("strings", n, "longest", longest, "address", at, flush=True)
    S = W.from_list(_strings(rng, n, longest, 256))
    chars, offs = np.asarray(S.chars), np.asarray(S.offsets)
    buf = torch.zeros(at + len(chars) + 1, dtype=torch.uint8, device="cuda")
    buf[at:at + len(chars)] = torch.from_numpy(chars.copy()).cuda()
    d = (buf[at:at + len(chars)], torch.from_numpy(offs.astype(np.int32)).cuda())
    pj = O.self_join_pj(S, 1)
    got = P.pj_self_join(d, 1)
    st = P.pj_last_stats()
    got = got.cpu().numpy() if hasattr(got, "cpu") else got
    assert np.array_equal(got, pj.pairs)
    assert (st["selected"], st["candidates"]) == (pj.selected, pj.candidates)


# one wide pass: tiles of 4096 ids from 2^18 on
@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 4097])
def test_large_sets(n):
    rng = np.random.default_rng(n)
    print("strings", n, flush=True)
    lens = rng.integers(5, 60, size=n)
    chars = rng.integers(0, 256, size=int(lens.sum())).astype(np.uint8).tobytes()
    at = np.concatenate([[0], np.cumsum(lens)])
    strings = [chars[at[k]:at[k + 1]] for k in range(n)]
    for k in range(0, n - 1, 1000):
        strings[k + 1] = strings[k]
    S = W.from_list(strings)
    pj = O.self_join_pj(S, 1)
    assert len(pj.pairs) >= (n - 1) // 1000
    assert np.array_equal(P.pj_self_join(S, 1), pj.pairs)


# strings too short for the larger thresholds: the index at tau = 4 is empty, those below are not, and
# the symbol codes are the set's for all of them
@pytest.mark.parametrize("longest", [0, 1, 2, 4, 5])
def test_short_sets(longest):
    rng = np.random.default_rng(longest)
    strings = [bytes(97 + rng.integers(0, 3, size=int(ln)).astype(np.uint8))
               for ln in rng.integers(0, longest + 1, size=200)]
    S = W.from_list(strings)
    index = P.pj_build_index(S, 0, 4)
    for tau in range(5):
        assert np.array_equal(P.pj_query(index, S, np.full(S.n, tau)), O.join_pj(S, S, tau).pairs)
        assert np.array_equal(P.pj_self_join(S, tau), O.self_join_pj(S, tau).pairs)
    index.free()
