"""Long strings verified by furthest rows: every width of lanes a candidate takes (thresholds of a part
around 8, 16 and 32), agreeing runs around the 32 characters compared at a time, edits at the ends of
the parts, strings cut short or extended, runs of one character (many equally long diagonals), the last
strings of the arena, and first passes that decide nothing or everything.  Pairs, candidates and DP cells
equal the oracle's."""
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


def _check(strings, tau):
    S = W.from_list(strings)
    exp = O.self_join_pj(S, tau)
    got = P.pj_self_join(S, tau)
    st = P.pj_last_stats()
    assert np.array_equal(got, exp.pairs)
    assert (st["candidates"], st["cells"]) == (exp.candidates, exp.cells)
    R = W.from_list(strings[::3])
    exp = O.join_pj(R, S, tau)
    assert np.array_equal(P.pj_join(R, S, tau), exp.pairs)
    assert P.pj_last_stats()["cells"] == exp.cells


def _near(rng, n, lo, hi, most, symbols):
    sym = np.frombuffer(symbols, dtype=np.uint8)
    ed = W._Editor(rng, sym, np.full(len(sym), 1 / len(sym)))
    out = []
    for k in range(n):
        if k % 3:
            s = out[k - k % 3]
            kind = int(rng.integers(4))
            if kind == 0:
                s = ed.edit(s, int(rng.integers(0, most + 1)))
            elif kind == 1:                       # edits at the ends
                s = ed.edit(s[:20], int(rng.integers(0, 4))) + s[20:-20] + ed.edit(s[-20:], 2)
            elif kind == 2:
                s = s[int(rng.integers(0, most + 1)):]
            else:
                s = s + bytes(sym[rng.integers(0, len(sym), size=int(rng.integers(0, most + 1)))])
            out.append(s[:2047])
        else:
            out.append(bytes(sym[rng.integers(0, len(sym), size=int(rng.integers(lo, hi + 1)))]))
    return out


@pytest.mark.parametrize("first", [None, "1", "4096"])
@pytest.mark.parametrize("tau", [1, 6, 7, 8, 14, 15, 16, 17, 30, 31, 32])
def test_thresholds(tau, first, monkeypatch):
    if first:
        monkeypatch.setenv("PJ_LONG_PASSES", first)
    rng = np.random.default_rng(tau)
    print("tau", tau, "first pass", first, flush=True)
    _check(_near(rng, 120, 160, 700, tau + 2, b"abcdefgh"), tau)


@pytest.mark.parametrize("length", [129, 2015, 2047])
def test_runs(length):
    """One edit at a time, a step of the position through two compares' characters."""
    rng = np.random.default_rng(length)
    base = rng.integers(97, 123, size=length).astype(np.uint8).tobytes()
    strings = [base]
    for at in list(range(60, 100)) + [0, 1, length - 2, length - 1]:
        strings.append(base[:at] + b"-" + base[at + 1:])
        strings.append((base[:at] + base[at + 1:]))
        strings.append((base[:at] + b"-" + base[at:])[:2047])
    _check(strings, 3)


@pytest.mark.parametrize("tau", [4, 9, 20])
def test_one_symbol(tau):
    strings = [b"a" * n for n in range(200, 200 + 2 * tau)] + \
              [b"a" * k + b"b" + b"a" * (220 - k) for k in range(0, 221, 20)]
    _check(strings, tau)
