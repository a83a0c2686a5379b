"""Workloads of the query path whose speed is watched.

Each case is one thing that a program does with the library: open a graph,
encode its terms, answer one triple pattern, several patterns in one pass, a
join or a union of subquery results, a whole query, a stream of single queries
and a batch of queries.  The graphs follow the laws of `synth/graph.py`
(subjects Zipf 1.0 over n/10 IDs, predicates Zipf 1.2 over 1000, objects
Zipf 1.1 over n/5 IDs through a bijection), drawn on the GPU.  The seed names
the resources and orders the triples of a case's graph: the same queries then
bind other IDs at other positions, and results keep their sizes.  The query mix
follows `synth/batch.py` (1 to 6 patterns, stars and chains half and half,
selectivities log-uniform in [1e-6, 1e-1]).

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  a program's inputs and handles before the call
  run(state)           one pass, and its outputs
  work(case)           the bytes a pass cannot do without
  exact(case, seed)    the same outputs in plain torch
"""
from __future__ import annotations

import ctypes
import random
from types import SimpleNamespace

import numpy as np
import torch

OP_SCAN, OP_JOIN = 1, 2
N_PREDICATES = 1000
CHUNK = 1 << 25


def listed():
    return [
        # one pattern (?s p ?o) on a graph of the size of the repository's
        # "small" one: an interactive lookup, all launch and call latency
        {"name": "scan_small", "kind": "scan", "n": 100_000, "form": "p", "share": 0.02,
         "layout": False},
        # one pattern at about 1% on the "medium" graph
        {"name": "scan_medium", "kind": "scan", "n": 50_000_000, "form": "p", "share": 0.01,
         "layout": False},
        # the FILTER form on the "large" graph: every triple whose object lies
        # in an ID range that keeps about 5%, all three columns out
        {"name": "scan_range_large", "kind": "scan", "n": 500_000_000, "form": "range",
         "share": 0.05, "layout": False},
        # the keysArray search: 12 patterns in one call, an odd graph size
        {"name": "scan_multi", "kind": "multi", "n": 30_000_007, "k": 12},
        # the join of two subquery results on object = subject
        {"name": "join", "kind": "join", "n": 50_000_000, "left": 0.1, "right": 0.1,
         "how": "inner"},
        # the DISTINCT union of 8 subquery results
        {"name": "union_distinct", "kind": "union", "n": 40_000_003, "k": 8, "share": 0.01,
         "distinct": True},
        # a 3-pattern star on ?s as one query, on the TripleID array alone
        {"name": "query_star", "kind": "query", "n": 50_000_000, "shape": "star", "k": 3,
         "layout": False},
        # a 4-pattern chain over frequent predicates, as the large benchmark
        # graph's, on the TripleID array alone
        {"name": "query_chain", "kind": "query", "n": 200_000_000, "shape": "chain", "k": 4,
         "layout": False},
        # serving: 16 queries of the mix, each a call of its own, on the
        # predicate-partitioned layout
        {"name": "serve", "kind": "serve", "n": 100_000_000, "plans": 16},
        # a batch of 256 queries of the mix in one call, partitioned layout
        {"name": "batch", "kind": "batch", "n": 100_000_000, "plans": 256},
        # opening a graph for serving: load (checks, statistics) and partition
        {"name": "load", "kind": "load", "n": 50_000_000, "layout": True},
        # the dictionary: 200k triples of IRIs and literals to rows, and a
        # page of results back to strings
        {"name": "dictionary", "kind": "dict", "n": 200_000, "page": 5_000},
    ]


def _between(rng, lo, hi):
    """A whole number, log-uniform in [lo, hi], odd as often as even."""
    return int(round(lo * (hi / lo) ** rng.random()))


def _share(rng, lo, hi):
    return float("%.4g" % (lo * (hi / lo) ** rng.random()))


def draw(rng: random.Random):
    kind = rng.choice(["scan", "scan", "scan", "multi", "join", "union", "query", "serve", "batch",
                       "load", "dict"])
    if kind == "scan":
        n = _between(rng, 50_000, 300_000_000)
        form = rng.choice(["p", "p", "po", "range", "prange", "s"])
        return {"kind": kind, "n": n, "form": form, "share": _share(rng, 1e-3, 0.15),
                "layout": form != "range" and n < 100_000_000 and rng.random() < 0.3}
    if kind == "multi":
        return {"kind": kind, "n": _between(rng, 100_000, 60_000_000), "k": rng.randint(2, 16)}
    if kind == "join":
        return {"kind": kind, "n": _between(rng, 200_000, 60_000_000),
                "left": _share(rng, 2e-3, 0.12), "right": _share(rng, 2e-3, 0.12),
                "how": rng.choice(["inner", "inner", "left", "full"])}
    if kind == "union":
        return {"kind": kind, "n": _between(rng, 200_000, 60_000_000), "k": rng.randint(2, 12),
                "share": _share(rng, 1e-3, 0.02), "distinct": rng.random() < 0.8}
    if kind == "query":
        shape = rng.choice(["star", "chain"])
        return {"kind": kind, "n": _between(rng, 1_000_000, 150_000_000), "shape": shape,
                "k": rng.randint(2, 4), "layout": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": kind, "n": _between(rng, 1_000_000, 100_000_000),
                "plans": rng.randint(4, 24)}
    if kind == "batch":
        return {"kind": kind, "n": _between(rng, 1_000_000, 100_000_000),
                "plans": _between(rng, 32, 256)}
    if kind == "load":
        return {"kind": kind, "n": _between(rng, 20_000, 60_000_000),
                "layout": rng.random() < 0.5}
    return {"kind": kind, "n": _between(rng, 1_000, 250_000), "page": _between(rng, 100, 6_000)}


# ---------------------------------------------------------------------------
# inputs: plain torch and numpy, from the seed alone
# ---------------------------------------------------------------------------

def _uniform(j, column):
    """Numbers in [0, 1) from row numbers (the finaliser of SplitMix64)."""
    x = (j * 3 + column + 1) * -7046029254386353131
    x = (x ^ ((x >> 30) & 0x3FFFFFFFF)) * -4658895280553007687
    x = (x ^ ((x >> 27) & 0x1FFFFFFFFF)) * -7723592293110705685
    x ^= (x >> 31) & 0x1FFFFFFFF
    return ((x >> 11) & 0x1FFFFFFFFFFFFF).double() * 2.0 ** -53


def _zipf(j, column, n_ids, a):
    """Ranks in [1, n_ids] with P(r) close to r**-a (the inverse of its
    integral at uniform numbers)."""
    u = _uniform(j, column)
    if a == 1.0:
        r = torch.exp(u * float(np.log(n_ids + 1.0)))
    else:
        top = (n_ids + 1.0) ** (1.0 - a) - 1.0
        r = (u * top + 1.0) ** (1.0 / (1.0 - a))
    return r.to(torch.int64).clamp_(1, n_ids)


def _coprime(a, n):
    while np.gcd(a, n) != 1:
        a += 2
    return a


def _graph(n, seed):
    """(n, 3) int32 triples on the GPU, in the order the seed gives them."""
    n_s, n_o = max(16, n // 10), max(16, n // 5)
    step, mul = _coprime(1_000_000_007, n), _coprime(2_654_435_761, n_o)
    first = (int(seed) * 48_271 + 11) % n
    g = torch.empty((n, 3), dtype=torch.int32, device="cuda")
    for a in range(0, n, CHUNK):
        b = min(n, a + CHUNK)
        j = (torch.arange(a, b, device="cuda") * step + first) % n
        g[a:b, 0] = _zipf(j, 0, n_s, 1.0)
        g[a:b, 1] = _zipf(j, 1, N_PREDICATES, 1.2)
        # the bijection keeps the hub object from being the hub subject
        g[a:b, 2] = (_zipf(j, 2, n_o, 1.1) * mul + 12_345) % n_o + 1
    return g


NAMES = 256  # a resource's ID changes with the seed within blocks of this many


def _named(ids, seed):
    """Subject and object IDs under the seed's naming."""
    return ((ids - 1) ^ (int(seed) % NAMES)) + 1


def _rename(x, seed):
    """The triples and the constants asked for, under the seed's naming
    (ranges are whole blocks of IDs)."""
    for pos in (0, 2):
        x.g[:, pos] = _named(x.g[:, pos], seed)
    for p in getattr(x, "patterns", []):
        p.s = _named(p.s, seed) if p.s else 0
        p.o = _named(p.o, seed) if p.o else 0
    if hasattr(x, "queries"):
        x.queries = [(shape, [(p, _named(o, seed) if o else 0) for p, o in terms])
                     for shape, terms in x.queries]


def _pattern(s=0, p=0, o=0, vs=-1, vp=-1, vo=-1, range_pos=-1, lo=0, hi=0):
    return SimpleNamespace(s=int(s), p=int(p), o=int(o), vs=vs, vp=vp, vo=vo,
                           range_pos=range_pos, lo=int(lo), hi=int(hi))


def _predicate(hist, share, skip=()):
    """The predicate whose share of the triples is closest, in log scale."""
    want = np.log(share * hist.sum())
    for p in np.argsort(np.abs(np.log(np.maximum(hist, 0.5)) - want), kind="stable"):
        if p and int(p) not in skip:
            return int(p)
    return 1


def _histogram(g):
    return torch.bincount(g[:, 1], minlength=N_PREDICATES + 1).cpu().numpy()


def _object_range(g, share):
    """[lo, hi) over object IDs that keeps about `share` of the triples."""
    cum = torch.cumsum(torch.bincount(g[:, 2]), 0)
    n = g.shape[0]
    best = None
    for start in np.linspace(0.3, 0.7, 9):   # a hub can make one window too heavy
        at = torch.tensor([start * n, (start + share) * n], device="cuda").to(cum.dtype)
        lo, hi = (max(1, int(x)) for x in torch.searchsorted(cum, at))
        hi = max(hi, lo + 1)
        # whole blocks of IDs
        lo, hi = (lo - 1) // NAMES * NAMES + 1, -(-(hi - 1) // NAMES) * NAMES + 1
        hi = min(hi, (cum.numel() - 1) // NAMES * NAMES + 1)
        hi = max(hi, lo + NAMES)
        kept = int(cum[min(hi, cum.numel()) - 1]) - int(cum[lo - 1])
        off = abs(np.log(max(kept, 1) / (share * n)))
        if best is None or off < best[0]:
            best = (off, lo, hi)
    return best[1], best[2]


class _Slices:
    """The triples ordered by (predicate, subject), and the sizes of stars and
    chains (counts only), to choose queries of bounded size."""

    def __init__(self, g):
        key = (g[:, 1].long() << 32) | g[:, 0]
        key, order = torch.sort(key)
        self.s, self.o = (key & 0xFFFFFFFF).int(), g[:, 2][order]
        self.hist = _histogram(g)
        self.start = np.concatenate([[0], np.cumsum(self.hist)])
        self.n = g.shape[0]
        self.size = int(max(int(self.s.max()), int(self.o.max()))) + 1
        self.present = np.nonzero(self.hist)[0]
        self.counted = {}

    def rows(self, term):
        a, b = int(self.start[term[0]]), int(self.start[term[0] + 1])
        s, o = self.s[a:b], self.o[a:b]
        if term[1]:
            keep = o == term[1]
            s, o = s[keep], o[keep]
        return s, o

    def subjects(self, term):
        """The term's distinct subjects, and how many triples each has."""
        if term not in self.counted:
            ids, cnt = torch.unique_consecutive(self.rows(term)[0], return_counts=True)
            self.counted[term] = ids, cnt.double()
        return self.counted[term]

    def objects(self, p):
        if ("o", p) not in self.counted:
            self.counted["o", p] = torch.unique(self.rows((p, 0))[1], return_counts=True)
        return self.counted["o", p]

    def by_object(self, term):
        """The term's rows in object order, the distinct objects, and the last
        row of each (no hub object's sum is left to atomics)."""
        if ("b", term) not in self.counted:
            o, order = torch.sort(self.rows(term)[1], stable=True)
            ids, cnt = torch.unique_consecutive(o, return_counts=True)
            self.counted["b", term] = order, ids, torch.cumsum(cnt, 0) - 1
        return self.counted["b", term]

    def term(self, sigma, with_object, rng):
        """(predicate, object or 0) of about sigma * n triples."""
        share = self.hist[self.present] / self.n
        if sigma >= share.min() or not with_object:
            return int(self.present[np.argmin(np.abs(np.log(share) - np.log(sigma)))]), 0
        rare = self.present[np.argsort(share, kind="stable")[:60]]
        p = int(rng.choice(rare))
        ids, cnt = self.objects(p)
        off = torch.abs(torch.log(cnt.double()) - float(np.log(sigma * self.n)))
        near = ids[off <= off.min()]
        return p, int(near[int(rng.integers(0, near.numel()))])

    def prefixes(self, shape, terms, cap):
        """Rows after each join, in plan order; stops once one exceeds cap or
        is empty."""
        out, ids, w = [], None, None
        for i, t in enumerate(terms):
            if shape == "star":
                d, c = self.subjects(t)
                if ids is None:
                    ids, w = d, c
                elif d.numel() == 0:
                    w = torch.zeros(0, device=d.device)
                else:
                    at = torch.searchsorted(d, ids).clamp_(max=d.numel() - 1)
                    keep = d[at] == ids
                    ids, w = ids[keep], w[keep] * c[at[keep]]
                out.append(float(w.sum()))
            else:
                s, o = self.rows(t)
                c = torch.ones(s.numel(), dtype=torch.float64, device=s.device) \
                    if w is None else w[s]
                out.append(float(c.sum()))
                if i + 1 < len(terms) and out[-1] <= cap:
                    by_o, ids_o, last = self.by_object(t)
                    run = torch.cumsum(c[by_o], 0)[last]
                    w = torch.zeros(self.size, dtype=torch.float64, device=s.device)
                    w[ids_o.long()] = torch.diff(run, prepend=run.new_zeros(1))
            if out[-1] > cap or out[-1] == 0:
                break
        return out

    def query(self, rng, shape, k, sigmas, lo, hi, tries, first_object=False):
        """(shape, terms) whose joins all have at most hi rows, and whose
        result has at least lo rows where `tries` draws find one."""
        best = ("star", [self.term(1e-3, False, rng)])
        for _ in range(tries):
            sig = 10.0 ** rng.uniform(np.log10(sigmas[0]), np.log10(sigmas[1]), size=k)
            terms = [self.term(x, shape == "star" or i == k - 1, rng) for i, x in enumerate(sig)]
            if first_object:
                ids, cnt = self.objects(terms[0][0])
                terms[0] = (terms[0][0], int(ids[torch.argmax(cnt)]))
            pre = self.prefixes(shape, terms, hi)
            if max(pre) <= hi:
                best = (shape, terms)
                if len(pre) == k and pre[-1] >= lo:
                    break
        return best


def _mix(slices, count, rng):
    """Queries of the batched and serving mix."""
    out = []
    for _ in range(count):
        k = int(rng.integers(1, 7))
        shape = "star" if rng.random() < 0.5 else "chain"
        out.append(slices.query(rng, shape, k, (1e-6, 1e-1), 1, 1 << 21, 6))
    return out


def _plan(shape, terms):
    pats, ops = [], []
    for i, (p, o) in enumerate(terms):
        if shape == "star":
            pats.append(_pattern(p=p, o=o, vs=0, vo=-1 if o else i + 1))
        else:
            pats.append(_pattern(p=p, o=o, vs=i, vo=-1 if o else i + 1))
        ops += [OP_SCAN, i]
        if i:
            ops += [OP_JOIN, 0 if shape == "star" else i]
    return SimpleNamespace(patterns=pats, ops=ops)


def _terms_of(n, seed):
    """The terms of n triples, in reading order, as UTF-8 bytes."""
    rng = np.random.default_rng(n)
    n_s, n_o = max(16, n // 4), max(16, n // 2)
    s = (np.exp(rng.random(n) * np.log(n_s + 1.0))).astype(np.int64)
    p = (np.exp(rng.random(n) * np.log(51.0))).astype(np.int64)
    o = rng.integers(1, n_o + 1, n)
    lit = rng.random(n) < 0.3
    base = b"http://example.org/%02x/" % (int(seed) % NAMES)
    terms = []
    for a, b, c, is_lit in zip(s.tolist(), p.tolist(), o.tolist(), lit.tolist()):
        terms.append(base + b"resource/%d" % a)
        terms.append(base + b"ontology/property%d" % b)
        terms.append(b"\"v\xc3\xa9rit\xc3\xa9 %d\"@fr" % c if is_lit
                     else base + b"resource/%d" % c)
    return terms


def _inputs(case, seed):
    """What prepare() and exact() share: the data and the constants asked for."""
    kind = case["kind"]
    rng = np.random.default_rng([case["n"], 77])
    x = SimpleNamespace(kind=kind)
    if kind == "dict":
        x.terms = _terms_of(case["n"], seed)
        x.page = min(case["page"], case["n"])
        return x
    x.g = g = _graph(case["n"], seed)
    if kind == "scan":
        hist, share, form = _histogram(g), case["share"], case["form"]
        if form == "range":
            lo, hi = _object_range(g, share)
            x.patterns = [_pattern(vs=0, vp=1, vo=2, range_pos=2, lo=lo, hi=hi)]
        else:
            p = _predicate(hist, share)
            if form == "p":
                x.patterns = [_pattern(p=p, vs=0, vo=1)]
            elif form == "s":      # a subject's (p, o) pairs
                x.patterns = [_pattern(s=int((case["n"] // 10) ** rng.random()), vp=0, vo=1)]
            else:
                o = torch.sort(g[:, 2][g[:, 1] == p])[0]
                if form == "po":   # one of the predicate's objects
                    x.patterns = [_pattern(p=p, o=int(o[o.numel() // 3]), vs=0)]
                else:              # the predicate's triples, half of its objects
                    mid = int(o[o.numel() // 2])
                    x.patterns = [_pattern(p=p, vs=0, vo=1, range_pos=2, lo=1,
                                           hi=-(-mid // NAMES) * NAMES + 1)]
    elif kind == "multi":
        hist, x.patterns, used = _histogram(g), [], set()
        for j in range(case["k"]):
            p = _predicate(hist, 10.0 ** rng.uniform(-3.5, -1.3), used)
            used.add(p)
            x.patterns.append(_pattern(p=p, vs=0, vo=1))
    elif kind == "join":
        hist = _histogram(g)
        a = _predicate(hist, case["left"])
        b = _predicate(hist, case["right"], {a})
        x.patterns = [_pattern(p=a, vs=0, vo=1), _pattern(p=b, vs=1, vo=2)]
    elif kind == "union":
        hist, x.patterns, used = _histogram(g), [], set()
        for _ in range(case["k"]):
            p = _predicate(hist, case["share"], used)
            used.add(p)
            x.patterns.append(_pattern(p=p, vs=0, vo=1))
    elif kind == "query":
        slices = _Slices(g)
        if case["shape"] == "star":
            x.queries = [slices.query(rng, "star", case["k"], (2e-4, 5e-3), 1e3, 2e6, 20,
                                      first_object=True)]
        else:
            x.queries = [slices.query(rng, "chain", case["k"], (2e-2, 2e-1), 1e3, 1e7, 12)]
    elif kind in ("serve", "batch"):
        x.queries = _mix(_Slices(g), case["plans"], rng)
    _rename(x, seed)
    return x


# ---------------------------------------------------------------------------
# the library
# ---------------------------------------------------------------------------

_CTX = []


def _context():
    """The program's one context (one device, one stream)."""
    if not _CTX:
        from paper_1807_01409_amd import Context
        _CTX.append(Context(0))
    return _CTX[0]


class _Columns:
    """A table's columns as one (columns, rows) device array, without a copy;
    the array keeps the table alive."""

    def __init__(self, table, n, ptr, stride, k):
        self.table = table
        self.__cuda_array_interface__ = {"shape": (k, n), "typestr": "<i4", "version": 2,
                                         "strides": (stride, 4), "data": (ptr, False)}


def _columns(ctx, table):
    n, k, _ = table.info()
    if n == 0 or k == 0:
        return torch.empty((k, n), dtype=torch.int32, device="cuda")
    ptr = [table.column_ptr(c) for c in range(k)]
    step = ptr[1] - ptr[0] if k > 1 else 4 * n
    if step >= 4 * n and all(ptr[c] == ptr[0] + c * step for c in range(k)):
        return torch.as_tensor(_Columns(table, n, ptr[0], step, k), device="cuda")
    with torch.cuda.stream(ctx.stream):
        return torch.cat([torch.as_tensor(_Columns(table, n, q, 4 * n, 1), device="cuda")
                          for q in ptr])


class _Rows:
    """A graph's resident triples as an (n, 3) device array, without a copy."""

    def __init__(self, graph):
        self.graph = graph
        self.__cuda_array_interface__ = {"shape": (graph.n, 3), "typestr": "<i4", "version": 2,
                                         "strides": None, "data": (graph.device_ptr, False)}


def prepare(case, seed):
    x = _inputs(case, seed)
    ctx = _context()
    state = SimpleNamespace(kind=case["kind"], ctx=ctx)
    if x.kind == "dict":
        # a string column on the device: bytes and offsets
        off = np.zeros(len(x.terms) + 1, dtype=np.int64)
        off[1:] = np.cumsum([len(t) for t in x.terms])
        state.bytes = torch.from_numpy(np.frombuffer(b"".join(x.terms), dtype=np.uint8).copy()).cuda()
        state.offsets = torch.from_numpy(off).cuda()
        state.n, state.page = case["n"], x.page
        return state
    torch.cuda.synchronize()   # the triples are drawn on another stream than the context's
    if x.kind == "load":
        state.triples, state.layout = x.g, case["layout"]
        return state
    state.graph = ctx.load(x.g)
    x.g = None
    if case.get("layout") or x.kind in ("serve", "batch"):
        state.graph.partition()
    if x.kind == "scan":
        state.pattern = x.patterns[0]
    elif x.kind == "multi":
        state.patterns = x.patterns
    elif x.kind in ("join", "union"):
        state.tables = [ctx.scan(state.graph, p) for p in x.patterns]
        state.graph = None
        state.how = case.get("how")
        state.distinct = case.get("distinct")
    else:
        state.plans = [_plan(*q) for q in x.queries]
    ctx.synchronize()
    return state


def run(state):
    ctx, kind = state.ctx, state.kind
    if kind == "scan":
        return _columns(ctx, ctx.scan(state.graph, state.pattern))
    if kind == "multi":
        return [_columns(ctx, t) for t in ctx.scan_multi(state.graph, state.patterns)]
    if kind == "join":
        l, r = state.tables
        if state.how == "inner":
            return _columns(ctx, ctx.join(l, 1, r, 0))
        return _columns(ctx, ctx.join_outer(l, 1, r, 0, state.how))
    if kind == "union":
        return _columns(ctx, ctx.union(state.tables, state.distinct))
    if kind in ("query", "serve"):
        return [_columns(ctx, ctx.query(state.graph, p)) for p in state.plans]
    if kind == "batch":
        out = [_columns(ctx, t) for t in ctx.query_batch(state.graph, state.plans)]
        # one array of all results, column after column
        with torch.cuda.stream(ctx.stream):
            return {"shapes": np.array([list(t.shape) for t in out], dtype=np.int64),
                    "cells": torch.cat([c for t in out for c in t.unbind(0)])}
    if kind == "load":
        graph = ctx.load(state.triples)
        counts = [graph.count(1, p, p + 1) for p in range(1, 65)]
        counts += [graph.count(pos, 1, 1 << b) for pos in (0, 2) for b in range(1, 25)]
        out = {"rows": torch.as_tensor(_Rows(graph), device="cuda"),
               "counts": np.array(counts, dtype=np.int64)}
        if state.layout:
            graph.partition()
            out["first"] = _columns(ctx, ctx.scan(graph, _pattern(p=3, vs=0, vo=1)))
        return out
    return _encode_decode(state)


def _encode_decode(state):
    """tid_encode of a device string column, then tid_decode of a page of rows
    (the C calls, as a program with device buffers makes them)."""
    from paper_1807_01409_amd.tid import Dict, TidError
    ctx, n = state.ctx, state.n
    lib = ctx._lib
    rows = torch.empty(3 * n, dtype=torch.int32, device="cuda")
    handle = ctypes.c_void_p()
    st = lib.tid_encode(ctx.ptr, ctypes.c_void_p(state.bytes.data_ptr()), state.bytes.numel(),
                        ctypes.c_void_p(state.offsets.data_ptr()), n, 1,
                        ctypes.c_void_p(rows.data_ptr()), ctypes.byref(handle))
    if st != 0:
        raise TidError(st, "tid_encode")
    terms = Dict(ctx, handle)
    page = 3 * state.page
    off = np.zeros(page + 1, dtype=np.uint64)
    text = np.empty(64 * page, dtype=np.uint8)
    st = lib.tid_decode(ctx.ptr, terms._p, ctypes.c_void_p(rows.data_ptr()), page, 1,
                        off.ctypes.data_as(ctypes.c_void_p),
                        text.ctypes.data_as(ctypes.c_void_p), text.size)
    if st != 0:
        raise TidError(st, "tid_decode")
    count, size = terms.info()
    return {"rows": rows, "terms": count, "bytes": size, "offsets": off.astype(np.int64),
            "text": text[:int(off[-1])]}


# ---------------------------------------------------------------------------
# the bytes of a pass
# ---------------------------------------------------------------------------

def work(case):
    """Each input read once, each output written once (outputs whose size the
    inputs decide are taken at their usual size)."""
    kind, n = case["kind"], case["n"]
    if kind == "scan":
        form, share = case["form"], case["share"]
        kept = {"p": 8 * share, "prange": 4 * share, "po": 4e-3 * share, "s": 0.0,
                "range": 12 * share}[form] * n
        read = 12.0 * n
        if case["layout"] and form != "s":
            read = 8.0 * n * share
        return {"bytes": read + kept, "flops": 0}
    if kind == "multi":
        return {"bytes": 12.0 * n + 8.0 * n * 0.013 * case["k"], "flops": 0}
    if kind == "join":
        rows = n * (case["left"] + case["right"])
        out = 12.0 * n * case["left"] * case["right"] * 1.5
        return {"bytes": 8.0 * rows + out, "flops": 0}
    if kind == "union":
        return {"bytes": 16.0 * n * case["share"] * case["k"], "flops": 0}
    if kind == "query":
        share = 1e-3 * case["k"] if case["shape"] == "star" else 0.07 * case["k"]
        return {"bytes": 8.0 * n * share if case["layout"] else 12.0 * n, "flops": 0}
    if kind in ("serve", "batch"):
        # patterns share slices: no more than every predicate's once
        read = min(case["plans"] * 3.5 * 8.0 * n * 0.009, 8.0 * n)
        return {"bytes": read + case["plans"] * 1.2e6, "flops": 0}
    if kind == "load":
        return {"bytes": n * (24.0 + (24.0 if case["layout"] else 0.0)), "flops": 0}
    return {"bytes": 3.0 * n * (31 + 8 + 4) + 0.4 * n * 31 + 3.0 * case["page"] * 40, "flops": 0}


# ---------------------------------------------------------------------------
# the same outputs in plain torch
# ---------------------------------------------------------------------------

def _x_scan(g, pat):
    keep = torch.ones(g.shape[0], dtype=torch.bool, device=g.device)
    for pos, c in enumerate((pat.s, pat.p, pat.o)):
        if c:
            keep &= g[:, pos] == c
    if pat.range_pos >= 0:
        v = g[:, pat.range_pos]
        keep &= (v >= pat.lo) & (v < pat.hi)
    rows = g[keep]
    return [(v, rows[:, pos].to(torch.int64))
            for pos, v in enumerate((pat.vs, pat.vp, pat.vo)) if v >= 0]


def _x_sort(cols, distinct=False):
    if not cols or cols[0].numel() == 0:
        return cols
    order = torch.arange(cols[0].numel(), device=cols[0].device)
    for c in reversed(cols):
        order = order[torch.argsort(c[order], stable=True)]
    cols = [c[order] for c in cols]
    if distinct:
        new = torch.ones(order.numel(), dtype=torch.bool, device=order.device)
        new[1:] = torch.stack([c[1:] != c[:-1] for c in cols]).any(0)
        cols = [c[new] for c in cols]
    return cols


def _x_join(left, right, var, how="inner"):
    """Lists of (variable, column), joined on `var`."""
    lk, rk = dict(left)[var], dict(right)[var]
    rk, order = torch.sort(rk, stable=True)
    lo, hi = torch.searchsorted(rk, lk), torch.searchsorted(rk, lk, right=True)
    cnt = hi - lo
    li = torch.repeat_interleave(torch.arange(lk.numel(), device=lk.device), cnt)
    first = torch.cumsum(cnt, 0) - cnt
    ri = order[lo[li] + torch.arange(li.numel(), device=lk.device) - first[li]]
    out = [(v, c[li]) for v, c in left] + [(v, c[ri]) for v, c in right if v != var]
    if how in ("left", "full"):
        lone = cnt == 0
        more = [c[lone] for _, c in left]
        more += [torch.zeros_like(more[0]) for v, _ in right if v != var]
        out = [(v, torch.cat([c, m])) for (v, c), m in zip(out, more)]
    if how == "full":
        key = dict(right)[var]
        lone = ~torch.isin(key, lk)
        more = [key[lone] if v == var else torch.zeros_like(key[lone]) for v, _ in left]
        more += [c[lone] for v, c in right if v != var]
        out = [(v, torch.cat([c, m])) for (v, c), m in zip(out, more)]
    return out


def _x_query(g, shape, terms):
    plan = _plan(shape, terms)
    out = _x_scan(g, plan.patterns[0])
    for i, p in enumerate(plan.patterns[1:], 1):
        out = _x_join(out, _x_scan(g, p), 0 if shape == "star" else i)
    return _x_sort([c for _, c in out])


def exact(case, seed):
    x = _inputs(case, seed)
    if x.kind == "scan":
        return torch.stack([c for _, c in _x_scan(x.g, x.patterns[0])])
    if x.kind == "multi":
        return [torch.stack([c for _, c in _x_scan(x.g, p)]) for p in x.patterns]
    if x.kind == "join":
        l, r = (_x_scan(x.g, p) for p in x.patterns)
        return torch.stack(_x_sort([c for _, c in _x_join(l, r, 1, case["how"])]))
    if x.kind == "union":
        parts = [[c for _, c in _x_scan(x.g, p)] for p in x.patterns]
        cols = [torch.cat(c) for c in zip(*parts)]
        return torch.stack(_x_sort(cols, True) if case["distinct"] else cols)
    if x.kind in ("query", "serve"):
        return [torch.stack(_x_query(x.g, *q)) for q in x.queries]
    if x.kind == "batch":
        out = [_x_query(x.g, *q) for q in x.queries]
        return {"shapes": np.array([[len(t), t[0].numel()] for t in out], dtype=np.int64),
                "cells": torch.cat([c for t in out for c in t])}
    if x.kind == "load":
        g = x.g
        counts = [int((g[:, 1] == p).sum()) for p in range(1, 65)]
        counts += [int((g[:, pos] < 1 << b).sum()) for pos in (0, 2) for b in range(1, 25)]
        out = {"rows": g, "counts": np.array(counts, dtype=np.int64)}
        if case["layout"]:
            out["first"] = torch.stack([c for _, c in _x_scan(g, _pattern(p=3, vs=0, vo=1))])
        return out
    ids, rows = {}, []
    for t in x.terms:
        rows.append(ids.setdefault(t, len(ids) + 1))
    page = x.terms[:3 * x.page]
    return {"rows": torch.tensor(rows, dtype=torch.int64), "terms": len(ids),
            "bytes": sum(len(t) for t in ids),
            "offsets": np.concatenate([[0], np.cumsum([len(t) for t in page])]).astype(np.int64),
            "text": np.frombuffer(b"".join(page), dtype=np.uint8)}
