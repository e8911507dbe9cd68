"""The list kernel that runs the parts' DPs as table reads (tau <= 4, indexed strings of up to 47
bytes), over every threshold of a part and length difference, lists of one lane to several segments,
strings at the edges (48 bytes take the banded kernel, probes 4 bytes longer than the longest indexed
string, part starts and lengths around the 4, 8 and 16 characters read at a time, the high word of
the position masks), exact and hashed keys, joins and batches with a tau per query.  Pairs, candidates
and DP cells equal the oracle's."""
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


@pytest.fixture(autouse=True)
def _lists(monkeypatch):
    monkeypatch.setenv("PJ_BUCKET_MIN_CANDIDATES", "0")     # every hit is bucketed


def _families(rng, n, lo, hi, tau, symbols):
    """Strings around a few stems, so that lists are long: a stem's copies have their ends redrawn
    or are edited anywhere."""
    sym = np.frombuffer(symbols, dtype=np.uint8)
    ed = W._Editor(rng, sym, np.full(len(sym), 1 / len(sym)))
    stems = [bytes(sym[rng.integers(0, len(sym), size=int(ln))])
             for ln in rng.integers(lo, hi + 1, size=4)]
    out = []
    for k in range(n):
        s = stems[int(rng.integers(len(stems)))]
        kind = int(rng.integers(3))
        if kind == 0:
            s = ed.edit(s, int(rng.integers(0, tau + 3)))
        else:
            cut = int(rng.integers(0, len(s) + 1))
            tail = bytes(sym[rng.integers(0, len(sym), size=max(len(s) - cut, 0))])
            s = s[:cut] + tail if kind == 1 else tail[:cut] + s[min(cut, len(tail)):]
        out.append(s[:hi])
    return out


def _check(strings, probes, tau):
    S, R = W.from_list(strings), W.from_list(probes)
    for what in ("self", "join"):
        if what == "self":
            pj, got = O.self_join_pj(S, tau), P.pj_self_join(S, tau)
        else:
            pj, got = O.join_pj(R, S, tau), P.pj_join(R, S, tau)
        st = P.pj_last_stats()
        assert np.array_equal(got, pj.pairs), what
        assert (st["candidates"], st["cells"]) == (pj.candidates, pj.cells), what


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("lo,hi", [(5, 9), (12, 16), (17, 24), (23, 28), (30, 40), (41, 47), (44, 48)])
def test_lengths(lo, hi, tau):
    rng = np.random.default_rng(1000 * hi + tau)
    print("lengths", lo, hi, "tau", tau, flush=True)
    strings = _families(rng, 700, lo, hi, tau, b"abc")
    probes = [s + b"abca"[:int(rng.integers(0, tau + 1))] for s in strings[:150]]
    _check(strings, probes, tau)


@pytest.mark.parametrize("symbols", [b"ab", bytes(range(97, 123)), bytes(range(256))])
@pytest.mark.parametrize("n", [64, 65, 129, 3000])
def test_lists(n, symbols):
    rng = np.random.default_rng(n + len(symbols))
    print("strings", n, "symbols", len(symbols), flush=True)
    strings = _families(rng, n, 14, 30, 3, symbols)
    _check(strings, strings[:60], 3)


def test_tau_per_query():
    rng = np.random.default_rng(5)
    strings = _families(rng, 3000, 8, 40, 4, b"abcd")
    asked = _families(rng, 10, 8, 40, 4, b"abcd") + strings[:600]
    taus = rng.integers(0, 5, size=len(asked)).astype(np.int32)
    index = P.pj_build_index(W.from_list(strings), 0, 4)
    got = P.pj_query(index, W.from_list(asked), taus)
    index.free()
    exp = []
    S = W.from_list(strings)
    for t in range(5):
        ids = np.flatnonzero(taus == t)
        pairs = O.join_pj(W.from_list([asked[k] for k in ids]), S, t).pairs
        exp.append(np.stack([ids[pairs[:, 0]], pairs[:, 1]], axis=1))
    exp = np.concatenate(exp)
    exp = exp[np.lexsort((exp[:, 1], exp[:, 0]))]
    assert np.array_equal(got, exp)
