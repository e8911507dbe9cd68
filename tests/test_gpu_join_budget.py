"""Small joins under memory budgets that held them before the probes had a position list and their
sorts and scans scratch of their own (the smallest budgets of that time, in bytes), and a join whose
hits reach the place that the list takes under a budget.  Pairs equal the oracle's."""
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


@pytest.mark.parametrize("gen, tau, budget", [
    (W.cfg2, 1, 177_408), (W.cfg2, 4, 216_832), (W.cfg2, 8, 365_824),
    (W.cfg3, 1, 165_632), (W.cfg3, 4, 193_536), (W.cfg3, 8, 298_496),
    (W.cfg4, 8, 681_216), (W.cfg4, 32, 2_171_392)])
def test_small_joins_fit(gen, tau, budget):
    S, R = gen(50, seed=50), gen(25, seed=51)
    print(gen.__name__, tau, budget, flush=True)
    assert np.array_equal(P.pj_join(R, S, tau, mem_budget=budget), O.join_bf(R, S, tau))
    with pytest.raises(P.PassJoinError) as ei:
        P.pj_join(R, S, tau, mem_budget=100_000)
    assert ei.value.code == P.PJ_ENOMEM


# equal letters: every selected substring is a hit, so the buffer of the Lemma 2 bound is full
@pytest.mark.parametrize("tau", [2, 16])
def test_hits_reach_the_list(tau):
    S = W.from_list([b"a" * n for n in range(130, 150)])
    exp = O.self_join_pj(S, tau)
    for budget in (0, 1 << 28):
        got = P.pj_self_join(S, tau, mem_budget=budget)
        st = P.pj_last_stats()
        assert np.array_equal(got, exp.pairs)
        assert (st["selected"], st["candidates"]) == (exp.selected, exp.candidates)
