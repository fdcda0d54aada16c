"""Performance cases of the framework: the work a user's program has it do.

Two servers' path: a client's query over a secret-shared attributed graph (open
the masked values, evaluate every predicate, AND them, join the edges), with the
dealer's keys made in the pass or given beforehand, alone, in a batch, or as
each server's own half in rounds.  Three servers' path: the paper's secEval,
secShuffle, secFetch, secAccess, the encoding of posting lists and the whole
secMatch.  A case is a dict of plain values; ``prepare`` makes what a program
holds before the call (shares, keys or tokens, plans, output buffers), ``run``
is one pass through the package's entry points, and ``work`` counts what the
path cannot do without.

Output buffers whose tail a call leaves unwritten (records beyond the opened
count) are zeroed once in ``prepare``.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2209_03526_amd import fss, secmatch
from paper_2209_03526_amd.runner import ChunkedRunner, QueryJob

DEALER_SEED = 20220903
PRF_KEYS = (41, 42, 43)
SHUFFLE_SEEDS = (101, 202, 303)

# 32-bit integer operations of one block of each cipher: AES-128 as table
# lookups (16 lookups and 16 XORs in each of 10 rounds), ChaCha12 by its
# definition (12 rounds of 4 quarter rounds of 12 operations, 16 final adds).
AES_OPS = 320
CHACHA_OPS = 12 * 4 * 12 + 16

# Predicates of a query: (target, kind, column).  Targets below the number of
# query vertices are vertex tables, the rest query edges.
FILTER = ((0, "eq", "label"), (0, "eq", "label"), (0, "range", "zipf"), (0, "range", "zipf"))
ONE_HOP = ((0, "eq", "label"), (1, "range", "attr"), (2, "eq", "elabel"))
TWO_HOP = ((0, "eq", "label"), (1, "range", "zipf"), (2, "eq", "label"), (2, "range", "zipf"), (3, "eq", "elabel"),
           (4, "range", "weight"))
PREDS = {0: FILTER, 1: ONE_HOP, 2: TWO_HOP}


def listed():
    return [
        # the smallest whole query: a 1,024-vertex random graph, one hop, the dealer's
        # masks and keys made for it; launches and latency
        {"name": "query_er_1k", "kind": "query", "hops": 1, "vertices": 1024, "edges": 8192, "dealt": True},
        # vertex filtering of one candidate table as large as the paper's largest
        # (10,000 candidates), the client's token given
        {"name": "filter_10k", "kind": "query", "hops": 0, "vertices": 10000, "edges": 0, "dealt": False},
        # an ordinary query: as many vertices as the paper's ego-network graph, an odd
        # number of edges, a two-hop path, masks and keys made for it
        {"name": "query_ego", "kind": "query", "hops": 2, "vertices": 107614, "edges": 999983, "dealt": True},
        # the largest: a two-hop path over 2^20 vertices and 2^23 edges, token given
        {"name": "query_2p23", "kind": "query", "hops": 2, "vertices": 1 << 20, "edges": 1 << 23, "dealt": False},
        # both servers of a deployment, each running its own half in rounds and
        # reading the other's message; token given
        {"name": "rounds_50k", "kind": "rounds", "hops": 2, "vertices": 50021, "edges": 400009},
        # a serving batch: 16 uneven queries, keys dealt and evaluated in waves that
        # fit a memory budget
        {"name": "batch_16", "kind": "batch", "queries": 16, "min_rows": 4096, "max_rows": 524288},
        # the paper's secEval: one range predicate over 300,007 candidates' one-hot
        # attributes of 2,000 positions, three servers, bits re-shared
        {"name": "sec_eval", "kind": "sec_eval", "candidates": 300007, "positions": 2000, "range": True},
        # secShuffle of a large table: 2^22 records of 64 bytes
        {"name": "shuffle_4m", "kind": "shuffle", "records": 1 << 22, "words": 16},
        # secFetch Case II over an ordinary candidate table: an odd number of records of
        # an odd width {bit || id || value}
        {"name": "fetch_100k", "kind": "fetch", "mode": "many", "records": 100003, "words": 21},
        # secAccess: the neighbours of 8 kept vertices among 30,011 candidates, 8,000
        # neighbour IDs (1,000-byte one-hot records)
        {"name": "access_8", "kind": "access", "candidates": 30011, "ids": 8000, "longest": 24, "matched": 8},
        # the data owner's upload: posting lists of 30,011 vertices over 16,384 IDs
        {"name": "encode_30k", "kind": "encode", "candidates": 30011, "ids": 16384, "longest": 24},
        # the paper's whole secMatch: a path over three vertex types
        {"name": "sec_match", "kind": "sec_match", "users": 200, "people": 8000, "companies": 1000, "friends": 40},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "query", "rounds", "batch", "sec_eval", "shuffle", "fetch", "access", "encode",
                       "sec_match"])
    if kind == "query":
        hops, dealt = rng.choice([0, 1, 2]), rng.random() < 0.5
        v = _log(rng, 1000, 1 << (18 if dealt else 20))
        return {"kind": kind, "hops": hops, "vertices": v, "edges": _log(rng, 4 * v, 8 * v) if hops else 0,
                "dealt": dealt}
    if kind == "rounds":
        v = _log(rng, 1000, 1 << 18)
        return {"kind": kind, "hops": rng.choice([1, 2]), "vertices": v, "edges": _log(rng, 4 * v, 8 * v)}
    if kind == "batch":
        return {"kind": kind, "queries": rng.randint(2, 24), "min_rows": _log(rng, 1000, 8000),
                "max_rows": _log(rng, 16000, 524288)}
    if kind == "sec_eval":
        return {"kind": kind, "candidates": _log(rng, 1000, 1 << 20), "positions": _log(rng, 16, 4096),
                "range": rng.random() < 0.5}
    if kind == "shuffle":
        return {"kind": kind, "records": _log(rng, 300, 1 << 21), "words": _log(rng, 2, 32)}
    if kind == "fetch":
        return {"kind": kind, "mode": rng.choice(["many", "valid", "unique"]), "records": _log(rng, 300, 1 << 21),
                "words": _log(rng, 2, 32)}
    if kind in ("access", "encode"):
        c = {"kind": kind, "candidates": _log(rng, 500, 1 << 16), "ids": _log(rng, 300, 16384),
             "longest": rng.randint(4, 32)}
        if kind == "access":
            c["matched"] = rng.randint(1, 16)
        return c
    return {"kind": kind, "users": _log(rng, 100, 300), "people": _log(rng, 500, 8000), "companies": _log(rng, 100, 1000),
            "friends": rng.randint(10, 40)}


# --------------------------------------------------------------------------- inputs

class _Inputs:
    """Values of one case, drawn on the GPU from its seed."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(int(seed) % (1 << 62) + 1)
        self.np = np.random.default_rng(int(seed) + 1)

    def words(self, n):
        """n uniform 32-bit words (shares, masks)."""
        return torch.randint(-2**31, 2**31, (max(1, n),), dtype=torch.int32, device=self.dev, generator=self.g)

    def below(self, bound, n):
        return torch.randint(0, bound, (max(1, n),), dtype=torch.int32, device=self.dev, generator=self.g)

    def uniform(self, n):
        return torch.rand((max(1, n),), dtype=torch.float64, device=self.dev, generator=self.g)

    def column(self, name, n):
        """Plain attribute values: labels, 20-bit numbers, 16-bit weights, or Zipf(1.1) ranks over 32 bits."""
        if name == "zipf":
            u = self.uniform(n).clamp_min_(1e-9)
            k = torch.floor(u.pow_(-10.0)).sub_(1.0).remainder_(4294967296.0)
            return torch.where(k >= 2147483648.0, k - 4294967296.0, k).to(torch.int32)
        return self.below({"label": 64, "attr": 1 << 20, "elabel": 4, "weight": 1 << 16}[name], n)

    def bounds(self, kind, name):
        """A predicate's constants: (a, 0) for equality, [lo, hi) for a range of a quarter to a half of the values."""
        if kind == "eq":
            return int(self.np.integers(0, {"label": 64, "elabel": 4}[name])), 0
        if name == "zipf":
            return int(self.np.integers(10, 30)), int(self.np.integers(1 << 20, 1 << 30))
        top, width = {"attr": (1 << 20, 1 << 18), "weight": (1 << 16, 1 << 14)}[name]
        lo = int(self.np.integers(0, top - width))
        return lo, lo + width

    def endpoints(self, n_vertices, n_edges):
        """Edge endpoints of a power-law graph (weights (i + 1)^(-1/1.1)), no self loops."""
        ends = [(self.uniform(n_edges).pow_(11.0).mul_(n_vertices)).to(torch.int32).clamp_max_(n_vertices - 1)
                for _ in range(2)]
        loop = ends[0] == ends[1]
        ends[1] = torch.where(loop, (ends[1] + 1) % n_vertices, ends[1])
        return ends

    def zeros(self, n):
        return torch.zeros(max(1, n), dtype=torch.int32, device=self.dev)


class _Pred:
    """One predicate's table column in shares, its constants, and the buffers of its masked values and keys."""

    def __init__(self, inp, target, kind, column, rows, keys, index, masks=True):
        self.target, self.rows, self.index = target, rows, index
        self.kind = fss.EQ if kind == "eq" else fss.RANGE
        self.a, self.hi = inp.bounds(kind, column)
        x = inp.column(column, rows)
        self.x0 = inp.words(rows)
        self.x1 = x - self.x0
        self.r = inp.words(rows) if masks else inp.zeros(rows)
        self.xhat = inp.zeros(rows)
        self.keys = fss.KeyBatch(self.kind, 32, rows) if keys else None

    def deal(self, query_id):
        fss.fss_keygen(DEALER_SEED, query_id, self.index, self.a, self.hi, self.r, self.keys)

    def open(self):
        fss.fss_mask_open(self.x0, self.x1, self.r, self.xhat)


def _tables(inp, case, keys=True, masks=True):
    hops, v, e = case["hops"], case["vertices"], case["edges"]
    src, dst = inp.endpoints(v, e) if hops else (None, None)
    preds = [_Pred(inp, t, kind, col, v if t <= hops else e, keys, k, masks)
             for k, (t, kind, col) in enumerate(PREDS[hops])]
    return src, dst, preds


# --------------------------------------------------------------------------- a query, both servers

def _prepare_query(case, seed):
    inp = _Inputs(seed)
    s = SimpleNamespace(dealt=case["dealt"], query_id=7 + int(seed) % 1000)
    s.src, s.dst, s.preds = _tables(inp, case, masks=not case["dealt"])
    s.plan = fss.Plan(DEALER_SEED, s.query_id, case["hops"] + 1, case["vertices"], case["edges"],
                      [(p.target, p.keys, p.xhat) for p in s.preds], s.src, s.dst).allocate()
    if not case["dealt"]:
        for p in s.preds:
            p.deal(s.query_id)
    return s


def _run_query(s):
    for p in s.preds:
        if s.dealt:
            fss.fss_dealer_masks(DEALER_SEED, s.query_id, p.index, p.rows, p.r)
            p.deal(s.query_id)
        p.open()
    fss.match_query(s.plan)
    return s.plan.out


# --------------------------------------------------------------------------- each server's half, in rounds

def _prepare_rounds(case, seed):
    inp = _Inputs(seed)
    s = SimpleNamespace(query_id=5)
    s.src, s.dst, s.preds = _tables(inp, case)
    for p in s.preds:
        p.deal(s.query_id)
    s.plans = [fss.Plan(DEALER_SEED, s.query_id, case["hops"] + 1, case["vertices"], case["edges"],
                        [(p.target, p.keys, p.xhat) for p in s.preds], s.src, s.dst).allocate() for _ in range(2)]
    s.msgs = [[inp.zeros(w) for w in fss.match_rounds(s.plans[0])] for _ in range(2)]
    return s


def _run_rounds(s):
    for p in s.preds:
        p.open()
    last = len(s.msgs[0])
    for r in range(last + 1):
        for b in range(2):
            fss.match_query(s.plans[b], party_mask=b + 1, round=r, peer_msg=s.msgs[1 - b][r - 1] if r else None,
                            msg=s.msgs[b][r] if r < last else None)
    return [s.plans[b].out[b] for b in range(2)]


# --------------------------------------------------------------------------- a batch of queries

def _batch_shapes(case):
    """(hops, rows) of each query: sizes spread over the logarithm, shapes in turn."""
    n, lo, hi = case["queries"], math.log(case["min_rows"]), math.log(case["max_rows"])
    return [((i * 2 + 1) % 3, int(math.exp(lo + (hi - lo) * ((i * 0.6180339887) % 1.0)))) for i in range(n)]


def _prepare_batch(case, seed):
    inp = _Inputs(seed)
    s = SimpleNamespace(preds=[], jobs=[])
    for i, (hops, rows) in enumerate(_batch_shapes(case)):
        src, dst, preds = _tables(inp, {"hops": hops, "vertices": rows, "edges": rows if hops else 0}, keys=False)
        s.preds += preds
        s.jobs.append(QueryJob(DEALER_SEED, 1000 + i, hops + 1, rows, rows if hops else 0,
                               [dict(target=p.target, kind=p.kind, rows=p.rows, a_or_lo=p.a, hi=p.hi, r=p.r, xhat=p.xhat)
                                for p in preds], src, dst))
    s.runner = ChunkedRunner(4 << 30)
    return s


def _run_batch(s):
    for p in s.preds:
        p.open()
    s.runner.run(s.jobs)
    return [job.plan.out[b] for job in s.jobs for b in range(2)]


# --------------------------------------------------------------------------- secEval

def _words(bits):
    return (bits + 31) // 32


def _onehot_shares(inp, rows, bits, place):
    """Three binary shares of `rows` one-hot records (record-major): place[r] is the set bit, -1 for none."""
    w = _words(bits)
    plain = torch.zeros(rows * w, dtype=torch.int32, device=inp.dev)
    at = torch.arange(rows, device=inp.dev)[place >= 0]
    p = place[place >= 0].to(torch.int64)
    plain[at * w + p // 32] = torch.bitwise_left_shift(torch.ones_like(p), p % 32).to(torch.int32)
    a, b = inp.words(rows * w), inp.words(rows * w)
    return [a, b, plain ^ a ^ b]


def _prepare_sec_eval(case, seed):
    inp = _Inputs(seed)
    n, npos = case["candidates"], case["positions"]
    s = SimpleNamespace(n=n, npos=npos)
    w = _words(npos)
    place = inp.below(npos, n)
    rec = _onehot_shares(inp, n, npos, place)
    s.shares = [t.view(n, w).t().contiguous() for t in rec]           # word-major
    s.keys = fss.KeyBatch(fss.RANGE if case["range"] else fss.EQ, secmatch.domain_bits(npos), 3)
    fss.fss_keygen(DEALER_SEED, 9, 0, npos // 4, npos // 2, inp.zeros(3), s.keys)
    evals = {(p, r): inp.zeros(w) for p in range(2) for r in range(3)}
    s.reqs = [(p, s.keys, r, npos, t) for (p, r), t in evals.items()]
    s.terms = [(evals[(pa, ra)], evals[(pb, rb)], s.shares[ja], s.shares[jb])
               for (pa, ra, ja), (pb, rb, jb) in secmatch.SERVER_TERMS]
    s.x3 = [inp.zeros(_words(n)) for _ in range(3)]
    s.z3 = [inp.zeros(_words(n)) for _ in range(3)]
    return s


def _run_sec_eval(s):
    fss.fss_eval_all_batch(s.reqs)
    for (ea, eb, sa, sb), x in zip(s.terms, s.x3):
        fss.rss_sec_eval(s.n, s.npos, ea, eb, sa, sb, x)
    fss.rss_reshare(s.n, s.x3, PRF_KEYS, 3, s.z3)
    return s.x3 + s.z3


# --------------------------------------------------------------------------- secShuffle and secFetch

def _prepare_shuffle(case, seed):
    inp = _Inputs(seed)
    n = case["records"] * case["words"]
    return SimpleNamespace(rows=case["records"], words=case["words"], table=[inp.words(n) for _ in range(3)],
                           seeds=[t + int(seed) for t in SHUFFLE_SEEDS], out=[inp.zeros(n) for _ in range(3)])


def _run_shuffle(s):
    fss.rss_shuffle(s.rows, s.words, s.table, s.seeds, s.out)
    return s.out


def _prepare_fetch(case, seed):
    inp = _Inputs(seed)
    n, w, mode = case["records"], case["words"], case["mode"]
    s = SimpleNamespace(mode=mode, rows=n, words=w, seeds=[t + int(seed) for t in SHUFFLE_SEEDS])
    if mode == "unique":                                             # one candidate matches
        s.table = [inp.words(n * w) for _ in range(3)]
        place = int(inp.np.integers(0, n))
        a, b, c = inp.words(_words(n)), inp.words(_words(n)), inp.zeros(_words(n))
        c[place // 32] = 1 << (place % 32) if place % 32 < 31 else -2**31
        s.bits = [a, b, a ^ b ^ c]
        s.out = [inp.zeros(w) for _ in range(3)]
    elif mode == "valid":                                            # posting records, half of them dummies
        place = torch.where(inp.below(2, n) == 1, inp.below(32 * w, n), torch.full((n,), -1, device=inp.dev))
        s.table = _onehot_shares(inp, n, 32 * w, place)
        s.out = [inp.zeros(n * w) for _ in range(3)]
    else:                                                            # {bit || record}, about half match
        s.table = [inp.words(n * w) for _ in range(3)]
        s.out = [inp.zeros(n * (w - 1)) for _ in range(3)]
    s.pos, s.count = inp.zeros(n), inp.zeros(1)
    return s


def _run_fetch(s):
    if s.mode == "unique":
        fss.rss_fetch_unique(s.rows, s.words, s.bits, s.table, s.out)
        return s.out
    call = fss.rss_fetch_many if s.mode == "many" else fss.rss_compact_valid
    call(s.rows, s.words, s.table, s.seeds, s.out, s.pos, s.count)
    return s.out + [s.pos, s.count]


# --------------------------------------------------------------------------- posting lists and secAccess

def _degrees(n, longest):
    """n list lengths: the quantiles of Zipf(1.8) - 1 up to `longest`, so that every seed's table is as large."""
    k = np.arange(1, 1 << 16, dtype=np.float64) ** -1.8
    deg = np.searchsorted(np.cumsum(k) / np.sum(k), (np.arange(n) + 0.5) / n)
    deg = np.minimum(deg, longest).astype(np.int64)
    deg[-1] = longest
    return deg


def _posting(inp, case):
    """A candidate table's posting lists: short lists mostly, a few long ones, distinct IDs, groups of 4."""
    n, ids = case["candidates"], case["ids"]
    p = SimpleNamespace(n=n, ids=ids, wx=_words(ids))
    longest = min(case["longest"], ids)
    who = inp.np.permutation(n)
    deg = _degrees(n, longest)[who]
    padded, _ = fss.rss_group_k(deg.astype(np.uint32), (who % 2).astype(np.uint32), 4)
    adj_off = np.concatenate([[0], np.cumsum(deg)])
    off = np.concatenate([[0], np.cumsum(padded.astype(np.int64))])
    own = np.repeat(np.arange(n), deg)
    k = np.arange(adj_off[-1]) - adj_off[own]
    step = inp.np.integers(1, max(2, ids // longest), n)              # distinct IDs: first + k * step < first + ids
    adj = (inp.np.integers(0, ids, n)[own] + k * step[own]) % ids
    slot = (inp.np.integers(0, 1 << 30, n)[own] + k) % np.maximum(padded[own], 1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.uint32)).view(np.int32)).to(inp.dev)  # noqa: E731
    p.deg, p.nrec, p.lmax = deg, int(off[-1]), int(padded.max())
    p.d_off, p.d_adj_off, p.d_adj, p.d_slot = dev(off), dev(adj_off), dev(adj), dev(slot)
    p.post = [inp.zeros(p.nrec * p.wx) for _ in range(3)]
    return p


def _encode(p):
    fss.rss_enc_posting_lists(p.n, p.ids, p.d_adj_off, p.d_adj, p.d_slot, p.d_off, p.nrec, (71, 72), 4, p.post)


def _prepare_encode(case, seed):
    return _posting(_Inputs(seed), case)


def _run_encode(p):
    _encode(p)
    return p.post


def _prepare_access(case, seed):
    inp = _Inputs(seed)
    s = _posting(inp, case)
    _encode(s)
    m = case["matched"]
    kept = inp.np.choice(s.n, m, replace=False)
    kept[0] = int(np.argmax(s.deg))
    place = torch.from_numpy(kept).to(inp.dev)
    s.idm = [t.view(m, -1) for t in _onehot_shares(inp, m, s.n, place)]
    s.ptrs = [s.idm[i][c].data_ptr() for c in range(m) for i in range(3)]
    s.attr = [inp.words(s.ids * 2) for _ in range(3)]
    s.counters = [3 + 2 * c for c in range(m)]
    s.seeds = [900 + 3 * c + i for c in range(m) for i in range(3)]
    s.ids3 = [inp.zeros(m * s.lmax * s.wx) for _ in range(3)]
    s.attrs3 = [inp.zeros(m * s.lmax * 2) for _ in range(3)]
    s.rows, s.count = inp.zeros(m * s.lmax), inp.zeros(m)
    return s


def _run_access(s):
    fss.rss_sec_access_batch(s.n, s.ids, s.ptrs, s.d_off, s.lmax, s.post, 2, s.attr, PRF_KEYS, s.counters, s.seeds,
                             s.ids3, s.attrs3, s.rows, s.count)
    return s.ids3 + s.attrs3 + [s.rows, s.count]


# --------------------------------------------------------------------------- the whole secMatch

def _lists(rng, n, ids, most):
    """Per vertex up to `most` distinct neighbour IDs."""
    deg = rng.integers(0, min(most, ids) + 1, n)
    first, step = rng.integers(0, ids, n), rng.integers(1, max(2, ids // most), n)
    return [(f + s * np.arange(d)) % ids for f, s, d in zip(first, step, deg)]


def _np_shares(rng, place, bits):
    w = _words(bits)
    plain = np.zeros((place.size, w), np.uint32)
    plain[np.arange(place.size), place // 32] = np.uint32(1) << (place % 32).astype(np.uint32)
    a, b = (rng.integers(0, 1 << 32, plain.shape, dtype=np.uint32) for _ in range(2))
    return np.stack([a, b, plain ^ a ^ b])


def _prepare_sec_match(case, seed):
    rng, shape = np.random.default_rng(int(seed) + 1), np.random.default_rng(151)
    n = {"U": case["users"], "P": case["people"], "C": case["companies"]}
    domains = {("U", "city"): 40, ("P", "age"): 100, ("C", "industry"): 16}
    # one graph for all seeds up to its vertices' names, so that a query finds as much in each
    name = {t: rng.permutation(k) for t, k in n.items()}
    shares = {("id", t): _np_shares(rng, np.arange(k), k) for t, k in n.items()}
    for (t, a), dom in domains.items():
        value = np.empty(n[t], np.int64)
        value[name[t]] = shape.integers(0, dom, n[t])
        shares[("attr", t, a)] = _np_shares(rng, value, dom)
    adj = {}
    for pair, most in ((("U", "P"), case["friends"]), (("P", "C"), 3)):
        plain = _lists(shape, n[pair[0]], n[pair[1]], most)
        adj[pair] = [None] * len(plain)
        for v, to in enumerate(plain):
            adj[pair][name[pair[0]][v]] = np.sort(name[pair[1]][to]).astype(np.uint32)
    padded = secmatch.padded_lengths(adj, 2)
    slots = {}
    for pair, lists in adj.items():
        turn = rng.integers(0, 1 << 30, len(lists))
        slots[pair] = np.concatenate([(t + np.arange(len(a))) % max(int(p), 1)
                                      for t, a, p in zip(turn, lists, padded[pair])]).astype(np.uint32)
    target = lambda t, a, lo, hi: SimpleNamespace(vtype=t, attr=a, kind="range", a=0, lo=lo, hi=hi)  # noqa: E731
    targets = [target("U", "city", 3, 8), target("P", "age", 25, 60), target("C", "industry", 4, 8)]
    return SimpleNamespace(graph=secmatch.encode_graph(n, domains, shares, adj, slots, 2), first=900 + int(seed) % 100000,
                           query=SimpleNamespace(query_id=31, targets=targets, parent=lambda i: i - 1 if i else None))


def _run_sec_match(s):
    found = secmatch.sec_match(s.graph, s.query, DEALER_SEED, PRF_KEYS, 3, s.first)
    return [np.stack([np.stack(r[t]) for r in found]) if found else np.zeros((0, 3), np.uint32)
            for t in range(len(s.query.targets))]


# --------------------------------------------------------------------------- the cases' interface

_KINDS = {
    "query": (_prepare_query, _run_query),
    "rounds": (_prepare_rounds, _run_rounds),
    "batch": (_prepare_batch, _run_batch),
    "sec_eval": (_prepare_sec_eval, _run_sec_eval),
    "shuffle": (_prepare_shuffle, _run_shuffle),
    "fetch": (_prepare_fetch, _run_fetch),
    "access": (_prepare_access, _run_access),
    "encode": (_prepare_encode, _run_encode),
    "sec_match": (_prepare_sec_match, _run_sec_match),
}


def prepare(case, seed):
    state = _KINDS[case["kind"]][0](case, seed)
    state.kind = case["kind"]
    return state


def run(state):
    return _KINDS[state.kind][1](state)


def exact(case, seed):
    """Every output is a string of bits (shares, positions, counts): the same for every implementation, with
    no value in 64 bits to be near."""
    return None


def _query_work(hops, v, e, dealt, key_passes):
    """Both servers: shares in (and masks when they are not drawn here), keys moved, bits out."""
    nbytes = flops = 0
    for t, kind, _ in PREDS[hops]:
        rows = v if t <= hops else e
        walks, key = (1, 432) if kind == "eq" else (2, 872)
        nbytes += rows * ((8 if dealt else 12) + 2 * key * key_passes)
        blocks = 2 * 26 * walks                                       # both servers' walks
        if dealt:
            blocks += 1 + 2 * 26 * walks + 2 * walks + (walks > 1)    # mask, tree, roots, wrap share
        flops += rows * blocks * AES_OPS
    return nbytes + hops * e * 8 + 2 * max(hops, 1) * (e if hops else v) / 8, flops


def _shuffle_work(n, w):
    slices = n * ((w + 15) // 16)
    return 6 * 4 * n * w, (5 * slices + 3 * (n / 8)) * CHACHA_OPS


def work(case):
    kind = case["kind"]
    if kind == "query":
        nbytes, flops = _query_work(case["hops"], case["vertices"], case["edges"], case["dealt"], 2 if case["dealt"] else 1)
    elif kind == "rounds":
        nbytes, flops = _query_work(case["hops"], case["vertices"], case["edges"], False, 1)
    elif kind == "batch":
        parts = [_query_work(h, r, r if h else 0, True, 2) for h, r in _batch_shapes(case)]
        nbytes, flops = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif kind == "sec_eval":
        n, w = case["candidates"], _words(case["positions"])
        # each server reads its two shares; three servers
        nbytes = 6 * 4 * n * w + 9 * n / 8
        flops = 6 * 2 * n * w + 3 * (n / 512) * CHACHA_OPS
    elif kind == "shuffle":
        nbytes, flops = _shuffle_work(case["records"], case["words"])
    elif kind == "fetch":
        n, w = case["records"], case["words"]
        if case["mode"] == "unique":
            nbytes, flops = 3 * 4 * n * w + 3 * n / 8, 15 * n * w
        else:                                                         # half of the records are kept
            nbytes, flops = _shuffle_work(n, w)
            nbytes = 3 * 4 * n * w * 1.5
    elif kind == "encode":
        words = float(np.sum(_degrees(case["candidates"], case["longest"]))) * _words(case["ids"])
        nbytes, flops = 12 * words, 2 * (words / 16) * CHACHA_OPS
    elif kind == "access":
        w, m = _words(case["ids"]), case["matched"]
        words = float(np.sum(_degrees(case["candidates"], case["longest"]))) * w
        nbytes = 12 * words + 12 * case["ids"] * 2 + m * 12 * case["longest"] * (w + 2) / 2
        flops = m * (15 * words + (3 + 5) * case["longest"] * (w / 16) * CHACHA_OPS)
    else:
        u, p, c = case["users"], case["people"], case["companies"]
        pairs = ((u, p, case["friends"] / 2), (p, c, 1.5))
        nbytes = sum(12 * a * d * _words(b) for a, b, d in pairs) + 12 * sum(k * _words(k) for k in (u, p, c))
        flops = 15 * nbytes / 12 * u / 8                              # a selection per kept user over its lists
    return {"bytes": float(nbytes), "flops": float(flops)}
