"""A small pj_query batch whose accepted candidates or candidates exceed its buffers goes on from its
one upload and its one probe: pairs and counts equal pj_join's of the same sets, with strings
shorter than the thresholds in both, and thresholds of each query's own equal the oracle's."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = ("selected", "hits", "candidates", "cells", "accepted", "side_pairs", "pairs")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.load()
    yield


def _check(S, Q, tau):
    joined = P.pj_join(Q, S, tau)
    sj = P.pj_last_stats()
    index = P.pj_build_index(S, 0, tau)
    for _ in range(2):
        got = P.pj_query(index, Q, np.full(Q.n, tau, np.int32))
        st = P.pj_last_stats()
        assert np.array_equal(got, joined)
        assert [st[k] for k in COUNTS] == [sj[k] for k in COUNTS]
        assert st["ms_upload"] > 0            # the batch's upload, not the general path's
    index.free()
    return sj


@pytest.mark.parametrize("equal", [2731, 9000])
def test_accepted(equal):
    # equal strings are accepted once per slot (3 times); the short ones through the side path
    S = W.from_list([b"the quick brown fox"] * equal + [b"", b"a", b"ab"] * 20)
    Q = W.from_list([b"the quick brown fox", b"a", b"the quick brown box"])
    st = _check(S, Q, 2)
    print(st, flush=True)
    assert st["accepted"] > 8192


@pytest.mark.parametrize("tau, letters", [(4, 97), (3, 96)])
def test_candidates(tau, letters):
    rng = np.random.default_rng(tau)

    def words(n):
        return [bytes(rng.integers(97, 97 + 98 - letters + 1, size=int(ln)).astype(np.uint8))
                for ln in rng.integers(3, 8, size=n)]

    st = _check(W.from_list(words(9000)), W.from_list(words(200)), tau)
    print(st, flush=True)
    assert st["candidates"] > 1 << 20


def test_own_thresholds(monkeypatch, tmp_path):
    # the buffers' limit lowered, so that few candidates are too many; a cache file in the options
    rng = np.random.default_rng(8)
    S = W.cfg2(3000, seed=8)
    ed = W._Editor(rng, W.ALPHA27, W.english27_probs())
    base = S.as_list()
    Q = W.from_list([ed.edit(base[int(rng.integers(len(base)))], int(rng.integers(0, 4))) for _ in range(90)])
    taus = rng.integers(0, 4, size=Q.n).astype(np.int32)
    exp = np.array(sorted((q, s) for t in range(4) for q, s in O.join_bf(Q, S, t).tolist()
                          if taus[q] == t), np.int32).reshape(-1, 2)
    index = P.pj_build_index(S, 0, 3)
    cache = tmp_path / "tune.txt"
    cache.write_text("# passjoin tune cache v4\n")
    lib = P.load()
    for limit in ("1", "50", "100000"):
        monkeypatch.setenv("PJ_BUCKET_MIN_CANDIDATES", limit)
        assert np.array_equal(P.pj_query(index, Q, taus), exp), limit
        assert P.pj_last_stats()["ms_upload"] > 0
        opt = P._options(False, False, P.MODE_AUTO, 0, None, str(cache))
        m = P._Marshalled(Q)
        out = P.PjPairs()
        assert lib.pj_query(index.handle, C.byref(m.s), taus.ctypes.data,
                            C.byref(opt), C.byref(out)) == P.PJ_OK
        cols = [np.ctypeslib.as_array(C.cast(v, C.POINTER(C.c_int32)), (out.count,)) for v in (out.a, out.b)]
        got = np.stack(cols, 1)
        assert np.array_equal(got, exp)
        lib.pj_pairs_free(C.byref(out))
    index.free()
