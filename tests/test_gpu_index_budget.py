"""mem_budget_bytes of pj_build_index: the budget bounds what the index holds (whole blocks, as
pj_index_info reports them) and what the build keeps beside it, the uploaded strings and the sorted
keys.  A build that fits gives an index that answers as the oracle does."""
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


def _fits(col, lo, hi, budget):
    try:
        return P.pj_build_index(col, lo, hi, mem_budget=budget)
    except P.PassJoinError as e:
        assert e.code == P.PJ_ENOMEM
        return None


def _round(v):
    return (v + 255) // 256 * 256


@pytest.mark.parametrize("n, lo, hi", [(1, 0, 0), (40, 1, 3), (3_000, 2, 2), (60_000, 1, 2)])
def test_smallest_budget(n, lo, hi):
    col = W.cfg2(max(n, 2), seed=n).subset(np.arange(n))
    top = 1 << 30
    index = _fits(col, lo, hi, top)
    held = index.info()["device_bytes"]
    index.free()
    # uploads and, at one time, the keys of one threshold (none is shorter than hi + 1 here)
    aside = _round(4 * (n + 1)) + _round(int(col.offsets[-1]) + 16)
    keys = min(8 * n * (t + 1) for t in range(lo, hi + 1))
    least, most = 0, top
    while most - least > 256:
        mid = (least + most) // 512 * 256
        index = _fits(col, lo, hi, mid)
        if index is None:
            least = mid
        else:
            assert index.info()["device_bytes"] <= mid
            index.free()
            most = mid
    print("strings", n, "index", held, "smallest budget", most, flush=True)
    assert held + aside <= most <= held + aside + _round(8 * n * (hi + 1))
    assert most >= aside + keys
    index = _fits(col, lo, hi, most)
    Q = col.subset(np.arange(min(n, 20)))
    got = P.pj_query(index, Q, np.full(Q.n, hi, np.int32))
    assert np.array_equal(got, O.join_bf(Q, col, hi))
    index.free()


def test_reported_without_a_budget():
    # small arrays share a block of 256 KiB: the index holds it whole
    index = P.pj_build_index(W.from_list([b"abc", b"abd"]), 1, 1)
    assert index.info()["device_bytes"] >= 256 << 10
    index.free()
