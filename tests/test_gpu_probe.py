"""The probe kernels at the edges of what each takes: tiles of 64 strings of one length, the slot
sizes 32, 64 and 127 bytes, the strings from 128 bytes on that take a block each (prefix hashes,
positions from a list, more than 512 (length, slot) pairs), for self-joins and joins of two sets.
Pairs, candidates and selected substrings equal the oracle's."""
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


def _near(rng, lengths, tau, symbols=b"abcd"):
    """Strings of the given lengths, every second one an edited copy of the one before."""
    sym = np.frombuffer(symbols, dtype=np.uint8)
    ed = W._Editor(rng, sym, np.full(len(sym), 1 / len(sym)))
    out = []
    for k, ln in enumerate(lengths):
        if k % 2 and out:
            out.append(ed.edit(out[-1], int(rng.integers(0, tau + 2)))[:2047])
        else:
            out.append(bytes(sym[rng.integers(0, len(sym), size=ln)]))
    return out


def _check(strings, other, tau):
    S = W.from_list(strings)
    for what in ("self", "join"):
        if what == "self":
            pj, got = O.self_join_pj(S, tau), P.pj_self_join(S, tau)
        else:
            R = W.from_list(other)
            pj, got = O.join_pj(R, S, tau), P.pj_join(R, S, tau)
        st = P.pj_last_stats()
        assert np.array_equal(got, pj.pairs), what
        assert (st["selected"], st["candidates"]) == (pj.selected, pj.candidates), what


@pytest.mark.parametrize("count", [1, 63, 64, 65, 129, 2100])
def test_tile_counts(count):
    rng = np.random.default_rng(count)
    print("strings of one length", count, flush=True)
    strings = _near(rng, [12] * count, 2, b"abcdefgh")
    _check(strings, strings[:70], 2)


@pytest.mark.parametrize("tau", [0, 1, 3, 8])
@pytest.mark.parametrize("length", [31, 32, 33, 63, 64, 65, 126, 127, 128, 129])
def test_slot_sizes(length, tau):
    rng = np.random.default_rng(100 * length + tau)
    print("length", length, "tau", tau, flush=True)
    lengths = [length + int(d) for d in rng.integers(-2, 3, size=150)]
    _check(_near(rng, lengths, tau), _near(rng, lengths[:40], tau), tau)


# 16: one batch of 289 pairs; 22 (23^2 = 529) and 32: several batches; two sets double the lengths
@pytest.mark.parametrize("tau", [4, 16, 22, 32, 63])
@pytest.mark.parametrize("length", [128, 257, 1023, 1024, 1990])
def test_long_strings(length, tau):
    rng = np.random.default_rng(10 * length + tau)
    print("length", length, "tau", tau, flush=True)
    lengths = [min(length + int(d), 2047) for d in rng.integers(-1, 2, size=24)] + [2047]
    _check(_near(rng, lengths, tau, b"ab cdefg"), _near(rng, lengths[:10], tau, b"ab cdefg"), tau)
