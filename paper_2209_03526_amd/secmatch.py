"""The paper's whole secure matching protocol, Alg. 2 (secMatch), over its own
encoding, on the GPU: for a tree query over a typed graph (a path V_1 -> V_2
-> ... -> V_q, or targets each hanging off an earlier one, as Fig. 1's),
target by target

  secEval (Alg. 3: full-domain evaluations of the replicated token,
           `fss_eval_all_batch`; each server's two terms),
  the re-share of its three-out-of-three bits into RSS,
  secFetch Case II (Alg. 4: the table {x || id || d}; shuffle, open, keep),
           these three for all groups of the target at once
           (`rss_sec_fetch_groups`),
  secAccess (Alg. 6, `rss_sec_access_batch`) of every kept vertex's neighbours of
           the next target's type, over the k-grouped posting lists of Alg. 1
           (`rss_enc_posting_lists`).

All three servers are simulated on one device.  Every step runs in the
library's kernels; this module only orders the calls and reads the counts
that the opens of secFetch and secAccess reveal, two synchronisations per
target: one after all of the target's secFetch calls (their counts decide
how many secAccess calls follow), one after all of its secAccess calls (each
with its lmax-row capacity); between them the calls are enqueued back to
back.

Readings where Alg. 2 leaves the order open: a target's candidates are
grouped by the kept vertex (of its parent target) whose neighbours they are,
and secFetch runs once per group, so each kept vertex keeps its parent (the
final reorganisation into subgraphs needs that tie); targets run in index
order, and within a target every group's secEval, re-share and secFetch come
first (group order), then the secAccess calls of the kept vertices (group by
group, child target by child target);
re-shares take PRF counters in order from `counter0` (secEval's re-share one,
secAccess two); the s-th shuffle (secFetch's and secAccess's alike) takes the
seeds (seed0 + 3s, +1, +2); predicate i's token is made with pred = i; an
empty group takes no randomness.  A result is one kept vertex per target,
each in the group its parent's vertex made, as the three shares of each
target's one-hot ID record; the client reconstructs and drops results that
use a vertex twice.
"""
from __future__ import annotations

from dataclasses import dataclass, field

import numpy as np
import torch

from . import fss

# The token's replicated key pairs (Sec. V-C): server CS_1 holds (k_1^1, k_1^2),
# CS_2 (k_2^2, k_1^3), CS_3 (k_2^3, k_2^1); with the one-hot shares (<e>_i,
# <e>_{i+1}) each evaluates Eq. predEval's two terms.  Entries: (party of the
# key, replica j - 1, share index - 1) of each term.
SERVER_TERMS = (((0, 0, 0), (0, 1, 1)),
                ((1, 1, 1), (0, 2, 2)),
                ((1, 2, 2), (1, 0, 0)))


def words(bits: int) -> int:
    return (bits + 31) // 32


def _plus(base: int, steps) -> list:
    """base + steps (an array of whole numbers) modulo 2^64, as Python integers: seeds and counters are
    C integers, of which the library takes the low bits, and base may be any of them."""
    return (np.uint64(base % 2**64) + np.asarray(steps).astype(np.uint64)).tolist()


# Rows that one library call numbers: the rows of a record table with 32 bits, a
# call's own rows with 31.
ROW_SPAN, CALL_ROWS = 1 << 32, (1 << 31) - 1


def _row_runs(base, n):
    """Runs (lo, hi) of consecutive groups (rows base[g] .. base[g] + n[g] - 1, base increasing) that one
    `rss_sec_fetch_groups` call takes: rows within ROW_SPAN of the run's first, at most CALL_ROWS in all."""
    if base[-1] + n[-1] - base[0] <= ROW_SPAN and n.sum() <= CALL_ROWS:
        return [(0, n.size)]
    runs, lo, rows = [], 0, 0
    for g in range(n.size):
        if g > lo and (base[g] + n[g] - base[lo] > ROW_SPAN or rows + n[g] > CALL_ROWS):
            runs.append((lo, g))
            lo, rows = g, 0
        rows += n[g]
    return runs + [(lo, n.size)]


def domain_bits(npos: int) -> int:
    """Input width of the token's keys for positions 0 .. npos - 1 (at least 8)."""
    return max(8, int(np.ceil(np.log2(max(npos, 2)))))


@dataclass
class EncodedGraph:
    """A typed graph as the servers hold it, resident on one device: per type
    its vertex count; per attribute its domain size; the three shares of the
    one-hot ID and attribute records (record-major, ceil(n/32) words each);
    per edge type (T, T2) the posting lists (CSR, k-grouped) and offsets."""
    n: dict
    domains: dict
    shares: dict = field(default_factory=dict)
    post: dict = field(default_factory=dict)
    off: dict = field(default_factory=dict)
    lmax: dict = field(default_factory=dict)


def _dev(a: np.ndarray, device):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).to(device)


def padded_lengths(adj: dict, k: int) -> dict:
    """Alg. 1's padded list lengths per edge type (T, T2): each vertex type's
    vertices grouped k at a time over the vector of their list lengths, list
    types in sorted order of the neighbour type (`rss_group_k_lists`)."""
    out = {}
    for t in sorted({p[0] for p in adj}):
        mine = sorted(p for p in adj if p[0] == t)
        lengths = np.array([[len(a) for a in adj[p]] for p in mine], np.uint32)
        padded, _ = fss.rss_group_k_lists(lengths, np.zeros(lengths.shape[1], np.uint32), k)
        for row, p in enumerate(mine):
            out[p] = padded[row]
    return out


def encode_graph(n: dict, domains: dict, shares: dict, adj: dict, slots: dict, k: int, split_keys=(1001, 1002),
                 counter: int = 4, device=None) -> EncodedGraph:
    """The data owner's upload: the one-hot RSS records of IDs and attributes
    (`shares`: {("id", T) | ("attr", T, name): (3, n_T, words) uint32}) moved
    to the device, and Alg. 1 for every edge type (T, T2) of `adj` (lists of
    neighbour IDs per vertex of T): each vertex type's vertices grouped k at a
    time over the vector of their list lengths (`rss_group_k_lists`), true
    IDs at the owner's slots (`slots[(T, T2)]`, flat in adjacency order),
    one-hot records split into RSS with the PRF (`rss_enc_posting_lists`)."""
    dev = device or torch.device("cuda")
    eg = EncodedGraph(dict(n), dict(domains))
    for key, sh in shares.items():
        eg.shares[key] = [_dev(sh[j].ravel(), dev) for j in range(3)]
    padded_of = padded_lengths(adj, k)
    for (t, t2), lists in sorted(adj.items()):
        lengths = np.array([len(a) for a in lists], np.uint32)
        padded = padded_of[(t, t2)]
        off = np.concatenate([[0], np.cumsum(padded, dtype=np.uint64)]).astype(np.uint32)
        adj_off = np.concatenate([[0], np.cumsum(lengths, dtype=np.uint64)]).astype(np.uint32)
        flat = np.concatenate([np.asarray(a, np.uint32) for a in lists]) if lengths.sum() else np.zeros(1, np.uint32)
        nrec = int(off[-1])
        wx = words(n[t2])
        out = [torch.empty(max(1, nrec * wx), dtype=torch.int32, device=dev) for _ in range(3)]
        d_off = _dev(off, dev)
        if nrec:
            fss.rss_enc_posting_lists(len(lists), n[t2], _dev(adj_off, dev), _dev(flat, dev),
                                      _dev(np.asarray(slots[(t, t2)], np.uint32) if lengths.sum() else flat, dev),
                                      d_off, nrec, split_keys, counter, out)
        eg.post[(t, t2)] = out
        eg.off[(t, t2)] = d_off
        eg.lmax[(t, t2)] = max(1, int(padded.max()) if padded.size else 1)
    torch.cuda.synchronize(dev)
    return eg


@dataclass
class _Target:
    """One target's groups of candidates: group g is rows base[g] .. of the
    one-hot records ids / vals (three device tensors each), n[g] of them, the
    neighbours of the kept vertex parent[g] = (group, kept row) of the parent
    target (None at target 0).  After secFetch: nkept[g] kept {id || d}
    records from row row0[g] of kept (one tensor: share, row, word)."""
    ids: list
    vals: list
    base: np.ndarray
    n: np.ndarray
    parent: list
    kept: torch.Tensor = None
    row0: np.ndarray = None
    nkept: np.ndarray = None


def sec_match(eg: EncodedGraph, query, tok_seed: int, prf_keys, counter0: int, seed0: int, device=None):
    """Alg. 2 for a tree query (``query.targets``: vertex type, attribute,
    predicate per target; ``query.parent(i)``: the target that target i hangs
    off, i - 1 for a path; readings in the module doc).  Returns the results,
    each a list over targets of the three shares (numpy uint32 records) of the
    target's one-hot ID."""
    dev = device or torch.device("cuda")
    counter, step = counter0, 0
    q = len(query.targets)
    children = [[c for c in range(1, q) if query.parent(c) == i] for i in range(q)]
    t0 = query.targets[0]
    one = lambda v: np.array([v], np.int64)  # noqa: E731
    targets = [None] * q
    targets[0] = _Target(eg.shares[("id", t0.vtype)], eg.shares[("attr", t0.vtype, t0.attr)], one(0),
                         one(eg.n[t0.vtype]), [None])
    zero3 = torch.zeros(3, dtype=torch.int32, device=dev)

    def empty(k):
        return torch.empty(max(1, k), dtype=torch.int32, device=dev)

    for i, tgt in enumerate(query.targets):
        st = targets[i]
        npos = eg.domains[(tgt.vtype, tgt.attr)]
        kb = fss.KeyBatch(fss.EQ if tgt.kind == "eq" else fss.RANGE, domain_bits(npos), 3, dev)
        fss.fss_keygen(tok_seed, query.query_id, i, tgt.a if tgt.kind == "eq" else tgt.lo, tgt.hi, zero3, kb)
        ev = {(party, rep): empty(words(npos)) for party in (0, 1) for rep in range(3)}
        fss.fss_eval_all_batch([(party, kb, rep, npos, t) for (party, rep), t in ev.items()])
        wi, wv = words(eg.n[tgt.vtype]), words(npos)
        rec = wi + wv
        # every group's secEval, re-share and secFetch, one library call (an
        # empty group takes no randomness)
        live = np.flatnonzero(st.n)
        base, n_live = st.base[live], st.n[live]
        total = int(n_live.sum())
        st.row0 = np.zeros(st.n.size, np.int64)
        st.row0[live] = np.cumsum(n_live) - n_live
        st.nkept = np.zeros(st.n.size, np.int64)
        st.kept = torch.empty((3, max(1, total), rec), dtype=torch.int32, device=dev)
        if live.size:
            fetched = empty(live.size)
            evals = [ev[(p, r)] for terms in SERVER_TERMS for p, r, _ in terms]
            b0, r0, ids, vals, out, cnt = 0, 0, st.ids, st.vals, st.kept.unbind(), fetched
            for lo, hi in _row_runs(base, n_live):
                if lo or base[-1] >= ROW_SPAN:   # the run's first group is row 0 of its call
                    b0, r0 = int(base[lo]), int(st.row0[live[lo]])
                    ids, vals = [t[b0 * wi:] for t in st.ids], [t[b0 * wv:] for t in st.vals]
                    out, cnt = [k[r0:] for k in st.kept], fetched[lo:]
                seeds = range(seed0 + 3 * (step + lo), seed0 + 3 * (step + hi))
                work = fss.rss_sec_fetch_groups((base[lo:hi] - b0).astype(np.uint32), n_live[lo:hi].astype(np.uint32),
                                                npos, evals, wi, ids, vals, prf_keys, counter + lo, seeds, out,
                                                empty(total - r0), cnt)
                del work                         # stream-ordered: reused only after the call's kernels
            counter += live.size
            step += live.size
            # the opens reveal how many candidates of each group match
            st.nkept[live] = fetched.cpu().numpy()
        # secAccess of every kept vertex of every group, for each child target:
        # call k (group by group, child by child) takes counter + 2k and
        # shuffle step + k; the calls of one child target go to the library as
        # one batch, and the validity opens' counts are read together
        nk = st.nkept
        first = len(children[i]) * (np.cumsum(nk) - nk)      # first call of each group
        base = st.kept.data_ptr() + 4 * st.kept[0].numel() * np.arange(3)
        opened = []
        for ci, c in enumerate(children[i]):
            nt = query.targets[c]
            pair = (tgt.vtype, nt.vtype)
            wx2, wv2 = words(eg.n[nt.vtype]), words(eg.domains[(nt.vtype, nt.attr)])
            lmax, nc = eg.lmax[pair], int(nk.sum())
            group = np.repeat(np.arange(nk.size), nk)
            r = np.arange(nc) - np.repeat(np.cumsum(nk) - nk, nk)
            k = first[group] + ci * nk[group] + r
            at = 4 * rec * (st.row0[group] + r)
            ids3, vals3 = [empty(nc * lmax * wx2) for _ in range(3)], [empty(nc * lmax * wv2) for _ in range(3)]
            cnt = empty(nc)
            if nc:
                idm = (base[None, :] + at[:, None]).ravel()
                seeds = _plus(seed0, (3 * (step + k)[:, None] + np.arange(3)[None, :]).ravel())
                work = fss.rss_sec_access_batch(eg.n[tgt.vtype], eg.n[nt.vtype], idm.tolist(), eg.off[pair], lmax,
                                                eg.post[pair], wv2, eg.shares[("attr", nt.vtype, nt.attr)], prf_keys,
                                                _plus(counter, 2 * k), seeds, ids3, vals3,
                                                empty(nc * lmax), cnt)
                del work
            targets[c] = _Target(ids3, vals3, np.arange(nc) * lmax, None,
                                 list(zip(group.tolist(), r.tolist())))
            opened.append((c, nc, cnt))
        calls = len(children[i]) * int(nk.sum())
        counter += 2 * calls
        step += calls
        for c, nc, cnt in opened:            # the first read waits for all of them
            targets[c].n = cnt.cpu().numpy()[:nc].astype(np.int64)
    return _results(targets, query, eg)


WHOLE_COPY = 1 << 18      # words of candidate records that _results copies as they are


def _results(targets, query, eg):
    """Every assignment of one kept vertex per target, each in the group its
    parent's vertex made (targets in index order), as host share records."""
    q = len(query.targets)
    out = []
    if not all(t.nkept.any() for t in targets):
        return out                           # some target keeps no vertex: no result, and nothing to copy
    # A target keeps few of its candidates, and its records are as wide as it has vertices / 32: the kept
    # rows' ID words are gathered on the device, group after group, and copied alone.  Up to WHOLE_COPY
    # words in all, one copy of everything costs less than the index and the gathers (100 users, 500 people,
    # 100 companies: 0.97 against 0.89 ms a query).
    first = [np.cumsum(st.nkept) - st.nkept for st in targets]       # each group's first kept row
    rows = [np.repeat(st.row0 - f, st.nkept) + np.arange(int(st.nkept.sum())) for st, f in zip(targets, first)]
    width = [words(eg.n[t.vtype]) for t in query.targets]
    whole = sum(st.kept.numel() for st in targets) <= WHOLE_COPY
    if whole:
        parts = [st.kept for st in targets]
    else:
        at = torch.from_numpy(np.concatenate(rows)).to(targets[0].kept.device).split([r.size for r in rows])
        parts = [st.kept[:, :, :w].index_select(1, r) for st, r, w in zip(targets, at, width)]
    flat = torch.cat([p.view(-1) for p in parts]).cpu().numpy().view(np.uint32)
    ends = np.cumsum([p.numel() for p in parts])
    ids = [f.reshape(p.shape) for f, p in zip(np.split(flat, ends[:-1]), parts)]
    if whole:
        ids = [f[:, r, :w] for f, r, w in zip(ids, rows, width)]
    groups_of = []                           # per target, the groups that a parent's kept vertex made
    for st in targets:
        of = {}
        for gi, p in enumerate(st.parent):
            of.setdefault(p, []).append(gi)
        groups_of.append(of)

    def walk(i, chosen):
        if i == q:
            out.append([[ids[t][j][first[t][gi] + r] for j in range(3)] for t, (gi, r) in enumerate(chosen)])
            return
        for gi in groups_of[i].get(None if i == 0 else chosen[query.parent(i)], []):
            for r in range(int(targets[i].nkept[gi])):
                walk(i + 1, chosen + [(gi, r)])

    walk(0, [])
    return out
