"""The memory of freed indexes serves later ones: indexes of changing sizes built, queried and freed
in turn, several held at a time, and from several threads at once, each on its own stream.  Results
equal the oracle's join, exactly."""
import threading

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


def _set(seed, n):
    rng = np.random.default_rng(seed)
    sym = np.frombuffer(b"abcdefgh", dtype=np.uint8)
    ed = W._Editor(rng, sym, np.full(len(sym), 1 / len(sym)))
    words = [bytes(sym[rng.integers(0, len(sym), size=int(ln))]) for ln in rng.integers(3, 40, size=n)]
    asked = [ed.edit(words[int(k)], int(rng.integers(0, 4))) for k in rng.integers(0, n, size=40)]
    return W.from_list(words), W.from_list(asked)


def _expected(S, Q, tau):
    return O.join_pj(Q, S, tau).pairs


# (smallest: every array shares a chunk; 64 KiB and 256 KiB steps; some MB)
SIZES = [1, 300, 3_000, 9_000, 40_000, 120_000]


def test_sizes_in_turn():
    for k, n in enumerate(SIZES + SIZES[::-1] + [SIZES[3]] * 6):
        print("strings", n, flush=True)
        S, Q = _set(k, n)
        with_two = [P.pj_build_index(S, 1, 2) for _ in range(2)]
        exp = _expected(S, Q, 2)
        for index in with_two:
            assert np.array_equal(P.pj_query(index, Q, np.full(Q.n, 2)), exp)
            index.free()


def test_threads():
    import torch
    cases = {(t, k): _set(100 * t + k, SIZES[(t + k) % 5]) for t in range(4) for k in range(5)}
    expected = {key: _expected(S, Q, 2) for key, (S, Q) in cases.items()}
    failed = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for k in range(5):
                    S, Q = cases[t, k]
                    index = P.pj_build_index(S, 1, 2, stream=stream)
                    got = P.pj_query(index, Q, np.full(Q.n, 2), stream=stream)
                    index.free()
                    if not np.array_equal(got, expected[t, k]):
                        failed.append((t, k, "pairs"))
        except Exception as e:                       # reported by the asserting thread
            failed.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not failed
