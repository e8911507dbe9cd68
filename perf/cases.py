"""Workloads of the join library: what its users have it do, through its public entry points.

  * self-joins of short (author names), medium (query log lines) and long (documents) string
    collections and of a small uniform one, from device arrays, as a captured plan, from host
    arrays, and in length windows;
  * a join of two sets held in host memory;
  * queries against a resident index: one at a time without allocation, in batches, in bulk, and
    as a stream of small requests through the server;
  * building an index and using it at once.

The collections have the shapes of the benchmark's: lengths, alphabets and near-duplicates as
stated at each generator below.  Every input is drawn on the GPU from the seed alone.

A case is a dict: kind (self, join, query, serve, build), text (uniform, short, medium, long,
served), n strings (the indexed set), m (the other set, the queries, or the requests of a served
stream), tau (of a join; an index holds 1 .. tau and queries draw theirs from it) and how (the
way the call is made).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1111_7171_amd as pj

# ------------------------------------------------------------------------------------------
# Collections
# ------------------------------------------------------------------------------------------

_LETTERS = b"abcdefghijklmnopqrstuvwxyz"
# English letter frequencies of a .. z; a space takes 0.18 of the text
_ENGLISH = (.082, .015, .028, .043, .127, .022, .020, .061, .070, .0015, .0077, .040, .024, .067,
            .075, .019, .00095, .060, .063, .091, .028, .0098, .024, .0015, .020, .00074)


def _zipf(m, s):
    return np.arange(1, m + 1, dtype=np.float64) ** -s


# text: shortest, longest string, share of near-duplicates, most edits of one, alphabet, weights
_TEXTS = {
    # half of the strings are copies of the other half with 0 .. 3 edits
    "uniform": (1, 24, 0.5, 3, _LETTERS + b" ", np.ones(27)),
    # lengths round(N(15, 4)), English frequencies
    "short": (5, 40, 0.3, 4, _LETTERS + b" ", np.array([.82 * p / sum(_ENGLISH) for p in _ENGLISH] + [.18])),
    # lengths round(N(45, 15)), 40 symbols with Zipf(1.1) frequencies
    "medium": (10, 120, 0.2, 8, _LETTERS + b"0123456789 .-_", _zipf(40, 1.1)),
    # lengths round(LogNormal(ln 700, 0.5)), words of a 20,000-word Zipf(1.0) vocabulary
    "long": (200, 2000, 0.1, 40, _LETTERS + b" ", np.ones(27)),
    # a serving index: lengths U{10 .. 120}, English frequencies, no near-duplicates
    "served": (10, 120, 0.0, 8, _LETTERS + b" ", np.array([.82 * p / sum(_ENGLISH) for p in _ENGLISH] + [.18])),
}
_MEAN_LEN = {"uniform": 14, "short": 15, "medium": 45, "long": 780, "served": 65}


class _Text:
    """Draws strings of one kind as padded rows on the GPU."""

    def __init__(self, text, gen):
        self.text, self.gen = text, gen
        self.lo, self.hi, self.dups, self.edits, symbols, weights = _TEXTS[text]
        self.symbols = torch.tensor(list(symbols), dtype=torch.uint8, device="cuda")
        self.cdf = torch.tensor(np.cumsum(weights)[:-1] / np.sum(weights), dtype=torch.float32, device="cuda")
        self.width = self.hi + 1

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.gen, device="cuda")

    def below(self, m):
        """One integer in [0, m) for each entry of m."""
        return torch.minimum((self.uniform(m.numel()) * m).long(), m - 1)

    def letters(self, *shape):
        return self.symbols[torch.bucketize(self.uniform(*shape), self.cdf, right=True)]

    def lengths(self, n, shortest=None):
        if self.text in ("uniform", "served"):
            lo = shortest or (8 if self.text == "uniform" else self.lo)
            hi = 20 if self.text == "uniform" else self.hi
            return lo + (self.uniform(n) * (hi - lo + 1)).long().clamp_(max=hi - lo)
        z = torch.randn(n, generator=self.gen, device="cuda")
        v = {"short": 15 + 4 * z, "medium": 45 + 15 * z, "long": 700 * torch.exp(0.5 * z)}[self.text]
        return v.round().long().clamp_(self.lo, self.hi)

    def rows(self, n, shortest=None):
        lens = self.lengths(n, shortest)
        if self.text != "long":
            return self.letters(n, self.width), lens
        return self.words(lens), lens

    def words(self, lens):
        """Rows of running text: each starts at a word of one long stream of words."""
        vocab = 20_000
        wlen = 3 + (self.uniform(vocab) * 11).long().clamp_(max=10)      # with its space
        wbase = torch.cumsum(wlen, 0) - wlen
        flat = self.symbols[(self.uniform(int(wlen.sum())) * 26).long().clamp_(max=25)]
        flat[wbase + wlen - 1] = 32
        p = _zipf(vocab, 1.0)
        cdf = torch.tensor(np.cumsum(p)[:-1] / p.sum(), dtype=torch.float32, device="cuda")
        at = torch.cumsum(lens + 13, 0) - (lens + 13)
        need = int(at[-1]) + self.width + 64
        ids = torch.bucketize(self.uniform(need // 4), cdf, right=True)
        ends = torch.cumsum(wlen[ids], 0)
        while int(ends[-1]) < need:
            ids = torch.cat([ids, ids])
            ends = torch.cumsum(wlen[ids], 0)
        ids = ids[: int(torch.searchsorted(ends, need)) + 1]
        ends = ends[: ids.numel()]
        begin = ends - wlen[ids]
        stream = torch.empty(int(ends[-1]), dtype=torch.uint8, device="cuda")
        for k in range(13):                                              # letter k of every word
            has = wlen[ids] > k
            stream[begin[has] + k] = flat[wbase[ids[has]] + k]
        first = begin[torch.searchsorted(begin, at)]
        col = torch.arange(self.width, device="cuda")
        return torch.cat([stream[(f[:, None] + col).clamp_(max=stream.numel() - 1)]
                          for f in first.split(8192)])

    def edit(self, rows, lens, k):
        """k[j] random edits of row j: a substitution, insertion or deletion at a uniform place
        (a substitution where the length would leave the collection's range)."""
        lo = min(self.lo, int(lens.min())) if lens.numel() else self.lo
        col = torch.arange(rows.shape[1], device="cuda")
        for e in range(int(k.max()) if k.numel() else 0):
            act = k > e
            op = self.below(torch.full_like(lens, 3))
            op = torch.where(((op == 1) & (lens >= self.hi)) | ((op == 2) & (lens <= lo)), 0, op)
            ins, cut = act & (op == 1), act & (op == 2)
            pos = self.below(torch.clamp(lens + ins.long(), min=1))
            sym = self.letters(lens.numel())
            src = col - (ins[:, None] & (col > pos[:, None])).long() + (cut[:, None] & (col >= pos[:, None])).long()
            rows = torch.gather(rows, 1, src.clamp_(max=rows.shape[1] - 1))
            put = act & ~cut & (lens + ins.long() > 0)
            rows[put.nonzero()[:, 0], pos[put]] = sym[put]
            lens = lens + ins.long() - cut.long()
        return rows, lens

    def collection(self, n, shortest=None):
        """n strings in random order, the kind's share of them edited copies of the others."""
        d = min(int(round(self.dups * n)), n - 1)
        rows, lens = self.rows(n - d, shortest)
        if d:
            src = self.below(torch.full((d,), n - d, device="cuda"))
            least = 0 if self.text == "uniform" else 1
            k = least + self.below(torch.full((d,), self.edits - least + 1, device="cuda"))
            r2, l2 = self.edit(rows[src], lens[src], k)
            rows, lens = torch.cat([rows, r2]), torch.cat([lens, l2])
        order = torch.randperm(n, generator=self.gen, device="cuda")
        return rows[order], lens[order]

    def queries(self, rows, lens, m, tau):
        """m strings with thresholds in 1 .. tau: every second one new, the others edited copies of
        the collection's strings with at most their threshold's edits."""
        taus = 1 + self.below(torch.full((m,), tau, device="cuda"))
        q, l = self.rows(m)
        src = self.below(torch.full((m,), lens.numel(), device="cuda"))
        r2, l2 = self.edit(rows[src], lens[src], 1 + self.below(taus))
        old = torch.arange(m, device="cuda") % 2 == 0
        return torch.where(old[:, None], r2, q), torch.where(old, l2, l), taus


def _flat(rows, lens):
    """Rows as the library takes them: all bytes back to back, and n + 1 offsets."""
    keep = torch.arange(rows.shape[1], device="cuda") < lens[:, None]
    offs = torch.zeros(lens.numel() + 1, dtype=torch.int64, device="cuda")
    offs[1:] = torch.cumsum(lens, 0)
    return rows[keep], offs.to(torch.int32)


def _host(strings):
    return tuple(t.cpu().numpy() for t in strings)


def _draw_sets(case, seed):
    """The case's indexed set, and its other set with thresholds, as rows."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    t = _Text(case["text"], gen)
    rows, lens = t.collection(case["n"], case.get("shortest"))
    other = t.queries(rows, lens, case["m"], case["tau"]) if case.get("m") else None
    return rows, lens, other


# ------------------------------------------------------------------------------------------
# Cases
# ------------------------------------------------------------------------------------------

def listed():
    return [
        # one name looked up as it is typed: latency, in a loop that must not allocate
        {"name": "query_one", "kind": "query", "text": "served", "n": 200_000, "m": 1, "tau": 4, "how": "noalloc"},
        # a request of a lookup service: 64 strings with thresholds of their own
        {"name": "query_batch", "kind": "query", "text": "served", "n": 500_000, "m": 64, "tau": 8, "how": "call"},
        # a file of new names matched against a name register
        {"name": "query_bulk", "kind": "query", "text": "short", "n": 400_000, "m": 20_011, "tau": 3, "how": "call"},
        # a service under load: 48 requests of 64 strings in flight on 4 slots
        {"name": "serve_stream", "kind": "serve", "text": "served", "n": 500_000, "m": 48 * 64, "tau": 8, "how": "server"},
        # the register changed: index it for every threshold again, then use it
        {"name": "build_index", "kind": "build", "text": "served", "n": 300_000, "m": 64, "tau": 4, "how": "call"},
        # a small list cleaned of near-duplicates
        {"name": "self_small", "kind": "self", "text": "uniform", "n": 10_000, "tau": 2, "how": "call"},
        # the benchmark's short strings at its lowest, a middle and its highest threshold; the
        # middle one as a job that repeats on the same data
        {"name": "self_short_t1", "kind": "self", "text": "short", "n": 1_000_000, "tau": 1, "how": "call"},
        {"name": "self_short_t2", "kind": "self", "text": "short", "n": 1_000_000, "tau": 2, "how": "plan"},
        {"name": "self_short_t4", "kind": "self", "text": "short", "n": 1_000_000, "tau": 4, "how": "call"},
        # two registers in host memory matched against each other
        {"name": "join_host", "kind": "join", "text": "short", "n": 400_000, "m": 50_021, "tau": 3, "how": "host"},
        # query log lines, and documents
        {"name": "self_medium_t6", "kind": "self", "text": "medium", "n": 500_000, "tau": 6, "how": "call"},
        {"name": "self_long_t16", "kind": "self", "text": "long", "n": 100_000, "tau": 16, "how": "call"},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["self", "self", "self", "self", "join", "query", "query", "serve", "build"])
    if kind == "self":
        text, most, taus = rng.choice([("uniform", 20_000, (1, 2, 3)), ("short", 1_000_000, (1, 2, 3, 4)),
                                       ("medium", 500_000, (2, 3, 4, 5, 6, 7, 8)),
                                       ("long", 100_000, (8, 12, 16, 24, 32))])
        c = {"kind": kind, "text": text, "n": _size(rng, 1000, most), "tau": rng.choice(taus),
             "how": rng.choice(["call", "call", "plan", "host", "streamed"])}
        if text == "uniform":
            c["shortest"] = rng.choice([1, 8])
        return c
    if kind == "join":
        text, most, taus = rng.choice([("short", 400_000, (1, 2, 3)), ("medium", 200_000, (2, 4, 6))])
        return {"kind": kind, "text": text, "n": _size(rng, 1000, most), "m": _size(rng, 500, most // 4),
                "tau": rng.choice(taus), "how": rng.choice(["host", "call"])}
    if kind == "query":
        how = rng.choice(["noalloc", "call", "call"])
        text, tau = rng.choice([("served", 8), ("served", 4), ("short", 3)])
        if how == "noalloc":
            tau = min(tau, 4)
        return {"kind": kind, "text": text, "n": _size(rng, 10_000, 500_000),
                "m": _size(rng, 1, 48 if how == "noalloc" else 20_000 if text == "short" else 1000),
                "tau": tau, "how": how}
    if kind == "serve":
        return {"kind": kind, "text": "served", "n": _size(rng, 20_000, 500_000), "m": 64 * rng.randint(8, 48),
                "tau": rng.choice([4, 8]), "how": "server"}
    return {"kind": kind, "text": rng.choice(["served", "short"]), "n": _size(rng, 10_000, 300_000),
            "m": _size(rng, 16, 256), "tau": rng.choice([2, 3, 4]), "how": "call"}


class _Served:
    """A server (which keeps its index alive), stopped when the program lets go of it."""

    def __init__(self, index):
        self.server = pj.Server(index, slots=4, max_batch_queries=512)

    def __del__(self):
        self.server.stop()


def prepare(case, seed):
    rows, lens, other = _draw_sets(case, seed)
    strings = _flat(rows, lens)
    kind, how = case["kind"], case["how"]
    s = {"case": case, "out": _room(case)}
    if kind == "self":
        s["strings"] = strings if how in ("call", "plan") else _host(strings)
        if how == "plan":
            s["plan"] = pj.Plan(strings, case["tau"])
        return s
    q, ql, taus = other
    queries = _flat(q, ql)
    if kind == "join":
        s["strings"], s["queries"] = (strings, queries) if how == "call" else (_host(strings), _host(queries))
        return s
    s["taus"] = taus.to(torch.int32).cpu().numpy()
    s["queries"] = _host(queries)
    if kind == "build":
        s["strings"] = _host(strings)
        return s
    s["index"] = pj.pj_build_index(_host(strings), 1, case["tau"])
    if kind == "serve":
        s["served"] = _Served(s["index"])
        chars, offs = s["queries"]
        s["requests"] = [((chars[offs[k]:offs[k + 64]], offs[k:k + 65] - offs[k]), s["taus"][k:k + 64])
                         for k in range(0, case["m"], 64)]
    return s


def _on_device(case):
    return case["kind"] in ("self", "join") and case["how"] in ("call", "plan")


def _room(case):
    """The program's result columns, with room for any seed's pairs (-1: unused): the next stage
    of such a program reads them where they are."""
    n, m, tau = case["n"], case.get("m", 0), case["tau"]
    if case["how"] == "noalloc":
        cap = 8192
    elif case["kind"] == "self":
        rate = {"uniform": 0.4 if case.get("shortest") == 1 else 0.01, "long": 0.0, "served": 0.0,
                "short": 1.5 * _CHANCE[min(tau, 4)], "medium": 1e-4 if tau > 6 else 1e-5}[case["text"]]
        cap = int(2 * n + rate * n * n / 2) + 10_000
    else:
        cap = 50_000 + m * (400 + int(n * 2e-5))
    if _on_device(case):
        return tuple(torch.full((cap,), -1, dtype=torch.int32, device="cuda") for _ in "ab")
    return tuple(np.full(cap, -1, dtype=np.int32) for _ in "ab")


class _Column:
    """One result column of a DevicePairs, for torch to read as it is."""

    def __init__(self, ptr, count):
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<i4", "data": (ptr, False), "version": 2}


def _keep(out, result):
    """Moves a call's pairs into the program's columns."""
    if isinstance(result, np.ndarray):
        count = len(result)
        out[0][:count], out[1][:count] = result[:, 0], result[:, 1]
    else:
        count = result.count
        if count:
            for column, ptr in zip(out, (result.raw.a, result.raw.b)):
                column[:count].copy_(torch.as_tensor(_Column(ptr, count), device="cuda"))
        result.free()
    return {"a": out[0], "b": out[1], "count": count}


def run(s):
    c, out = s["case"], s["out"]
    kind, how, tau = c["kind"], c["how"], c["tau"]
    if kind == "self":
        if how == "plan":
            return _keep(out, s["plan"].run())
        if how == "streamed":
            # windows of a quarter of the collection's bytes
            return _keep(out, pj.pj_self_join_streamed(s["strings"], tau, max(len(s["strings"][0]) // 4, 1)))
        return _keep(out, pj.pj_self_join(s["strings"], tau, outputs_on_device=how == "call"))
    if kind == "join":
        return _keep(out, pj.pj_join(s["queries"], s["strings"], tau, outputs_on_device=how == "call"))
    if kind == "serve":
        server = s["served"].server
        ids = [server.submit(q, t) for q, t in s["requests"]]
        got = [server.wait(i)[0] for i in ids]
        return dict(_keep(out, np.concatenate(got)), counts=np.array([len(g) for g in got]))
    if kind == "build":
        index = pj.pj_build_index(s["strings"], 1, tau)
        pairs = pj.pj_query(index, s["queries"], s["taus"])
        index.free()
        return _keep(out, pairs)
    if how == "noalloc":
        m = pj.pj_query_noalloc(s["index"], s["queries"], s["taus"], *out)
        return {"a": out[0], "b": out[1], "count": m}
    return _keep(out, pj.pj_query(s["index"], s["queries"], s["taus"]))


# Similar pairs by chance, per pair of short strings (the other kinds have about one per
# near-duplicate only)
_CHANCE = {1: 0.0, 2: 2e-7, 3: 8.8e-6, 4: 8.2e-5}


def work(case):
    """The strings read once (a query reads its own strings; its index is the program's) and the
    pairs written once.  The work is integer and no contraction: no flops are counted."""
    n, m, length = case["n"], case.get("m", 0), _MEAN_LEN[case["text"]]
    rate = _CHANCE[min(case["tau"], 4)] if case["text"] == "short" else 0.0
    read = (0 if case["kind"] in ("query", "serve") else n) * (length + 4) + m * (length + 8)
    if case["kind"] == "self":
        pairs = _TEXTS[case["text"]][2] * n + rate * n * n / 2
    else:
        pairs = 0.5 * m + rate * n * m
    return {"bytes": read + 8 * pairs, "flops": 0}


# ------------------------------------------------------------------------------------------
# The pairs by their definition
# ------------------------------------------------------------------------------------------

def _distances(a, la, b, lb):
    """Levenshtein distance of row k of a and row k of b, all cells of every row."""
    j = torch.arange(b.shape[1] + 1, device="cuda")
    d = j.repeat(a.shape[0], 1)
    done = torch.gather(d, 1, lb[:, None])[:, 0]
    for i in range(int(la.max()) if la.numel() else 0):
        step = torch.minimum(d[:, 1:] + 1, d[:, :-1] + (a[:, i:i + 1] != b))
        step = torch.cat([d[:, :1] + 1, step], 1)
        d = torch.cummin(step - j, 1).values + j
        done = torch.where(la == i + 1, torch.gather(d, 1, lb[:, None])[:, 0], done)
    return done


def exact(case, seed):
    """Every pair within the length difference, compared whole; for cases of up to 2 x 10^8
    pairs of short rows."""
    rows, lens, other = _draw_sets(case, seed)
    if case["kind"] == "self":
        q, ql, taus = rows, lens, torch.full_like(lens, case["tau"])
    else:
        q, ql, taus = other
        if case["kind"] == "join":
            taus = torch.full_like(taus, case["tau"])
    if ql.numel() * lens.numel() * rows.shape[1] > 5e9 or case["kind"] == "serve":
        return None
    found = []
    step = max(1, 4_000_000 // lens.numel())
    for k in range(0, ql.numel(), step):
        near = (ql[k:k + step, None] - lens).abs() <= taus[k:k + step, None]
        x, y = near.nonzero(as_tuple=True)
        x = x + k
        if case["kind"] == "self":
            x, y = x[x < y], y[x < y]
        for xs, ys in zip(x.split(1_000_000), y.split(1_000_000)):
            ok = _distances(q[xs], ql[xs], rows[ys], lens[ys]) <= taus[xs]
            found.append(torch.stack([xs[ok], ys[ok]], 1))
    pairs = torch.cat(found) if found else torch.empty(0, 2, dtype=torch.int64, device="cuda")
    pairs = pairs[torch.argsort(pairs[:, 0] * lens.numel() + pairs[:, 1])]
    a, b = (torch.as_tensor(column).to(torch.int64) for column in _room(case))
    count = len(pairs)
    a[:count], b[:count] = pairs[:, 0].to(a.device), pairs[:, 1].to(b.device)
    return {"a": a, "b": b, "count": count}
