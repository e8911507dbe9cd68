"""The first pass of rows of long strings (PJ_LONG_PASSES: its rows, the first of a comma list) around
the 64 rows whose characters are staged at a time: pairs, candidates and cells equal the oracle's for
any number of rows, and a list with a count out of range is refused."""
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


def _set(tau):
    rng = np.random.default_rng(700 + tau)
    return W.random_small(rng, 300, alphabet=b"abcd", lmin=140, lmax=700, dup_frac=0.6, kmax=tau + 2)


@pytest.mark.parametrize("tau", [5, 24])
def test_rows(tau, monkeypatch):
    col = _set(tau)
    exp = O.self_join_pj(col, tau)
    for rows in ("", "1", "31", "63", "64", "65", "127", "128", "129", "4096", "65,1"):
        print("tau", tau, "rows", rows, flush=True)
        monkeypatch.setenv("PJ_LONG_PASSES", rows)
        got = P.pj_self_join(col, tau)
        st = P.pj_last_stats()
        assert np.array_equal(got, exp.pairs), rows
        assert (st["candidates"], st["cells"]) == (exp.candidates, exp.cells), rows


@pytest.mark.parametrize("rows", ["0", "4097", "x", "8,0", "8,4097", ",8"])
def test_refused(rows, monkeypatch):
    monkeypatch.setenv("PJ_LONG_PASSES", rows)
    with pytest.raises(P.PassJoinError):
        P.pj_self_join(_set(5), 5)
