"""Evaluation and the dealer at the edges of their wave tiles (64 rows of an
equality or 32 of a range; 32 rows of one tree) and of their launch shapes (one
wave per workgroup up to 16), and full-domain
evaluation at the edges of its 128-point leaves: every share and key looked at
equals the oracle's, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, B, T, U
from keylayout import from_device
from oracle import fss as ofss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as lib
    return lib


def _rand_u32(seed, n):
    return np.random.default_rng(seed).integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


def _check(fss, kind, nbits, n):
    seed = 1234 + n
    top = (1 << nbits) - 1
    r, x = _rand_u32(seed, n), _rand_u32(seed + 1, n) & np.uint32(top)
    a, hi = (int(x[n // 2]), 0) if kind == 0 else sorted((int(x[0]), int(x[-1]) or 1))
    xhat = (x.astype(np.uint64) + r).astype(np.uint32)
    kb = fss.KeyBatch(kind, nbits, n)
    fss.fss_keygen(seed, 3, 1, a, hi, T(r), kb)
    rows = np.arange(n) if n <= 20000 else np.unique(np.concatenate(
        [np.arange(70), np.arange(n - 70, n), np.random.default_rng(n).integers(0, n, 3000)]))
    if kind == 0:
        keys = ofss.keygen_eq(nbits, seed, 3, 1, a, r[rows], rows=rows)
    else:
        keys = ofss.keygen_range(nbits, seed, 3, 1, a, hi, r[rows], rows=rows)
    run, ev = (fss.fss_eval_eq, ofss.eval_eq) if kind == 0 else (fss.fss_eval_lt, ofss.eval_range)
    nw = (n + 31) // 32
    recon = np.zeros(nw, np.uint32)
    for b in range(2):
        out = torch.full((nw + 3,), -1, dtype=torch.int32, device=DEV)
        run(b, kb, T(xhat), out)
        got = U(out)
        assert (got[nw:] == 0xFFFFFFFF).all()                 # nothing past the last word
        if n % 32:
            assert got[nw - 1] >> (n % 32) == 0               # pad bits
        want = ev(nbits, b, keys[b], xhat[rows])
        np.testing.assert_array_equal(ofss.unpack_bits(got[:nw], n)[rows], want)
        recon ^= got[:nw]
    truth = (x == a) if kind == 0 else ((x >= a) & (x < hi))
    np.testing.assert_array_equal(ofss.unpack_bits(recon, n), truth.astype(np.uint8))


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("nbits,n", [(32, 31), (32, 32), (32, 33), (8, 63), (32, 64), (12, 65), (32, 16383),
                                     (32, 16385), (32, 32769), (32, 300001)])
def test_eval_tile_edges(fss, kind, nbits, n):
    _check(fss, kind, nbits, n)


@pytest.mark.parametrize("kind,n", [(0, 15), (0, 17), (1, 7), (1, 9), (0, 131072), (0, 131073), (1, 65536), (1, 65537)])
def test_eval_quad_tile_edges(fss, kind, n):
    """Quad tiles (16 rows of an equality, 8 of a range; 2,048 wave tiles are the most that take them)."""
    _check(fss, kind, 32, n)


def test_eval_many_workgroups(fss):
    """2^21 + 33 range rows: 65,538 wave tiles, the last workgroup with two of them."""
    _check(fss, 1, 32, (1 << 21) + 33)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("nbits,npoints", [(8, 1), (8, 127), (8, 256), (9, 129), (16, 4097), (16, 33000), (17, 65537)])
def test_eval_all_leaf_edges(fss, kind, nbits, npoints):
    """A wave walks 64 leaves of an equality or 32 of a range, a workgroup four waves."""
    seed, row = 77 + npoints, 1
    r = np.zeros(3, np.uint32)
    a, hi = (1 << nbits) // 3, (1 << nbits) - 2
    kb = fss.KeyBatch(kind, nbits, 3)
    fss.fss_keygen(seed, 9, 0, a, hi if kind else 0, T(r), kb)
    keys = (ofss.keygen_range(nbits, seed, 9, 0, a, hi, r) if kind else ofss.keygen_eq(nbits, seed, 9, 0, a, r))
    ev = ofss.eval_range if kind else ofss.eval_eq
    xs = np.arange(npoints, dtype=np.uint32)
    nw = (npoints + 31) // 32
    for b in range(2):
        out = torch.full((nw + 3,), -1, dtype=torch.int32, device=DEV)
        fss.fss_eval_all(b, kb, row, npoints, out)
        want = ofss.pack_bits(ev(nbits, b, np.repeat(keys[b][row:row + 1], npoints, axis=0), xs))
        np.testing.assert_array_equal(U(out, nw), want)
        assert (U(out)[nw:] == 0xFFFFFFFF).all()


@pytest.mark.parametrize("kind,nbits,n", [(0, 32, 31), (0, 8, 33), (1, 32, 32), (1, 9, 33), (1, 32, 8193),
                                          (0, 32, 16417), (1, 32, 40000), (0, 32, 7), (1, 32, 9), (0, 32, 98304), (0, 32, 98305),
                                          (1, 32, 49152), (1, 32, 49153)])
def test_keygen_tile_edges(fss, kind, nbits, n):
    """The dealer's wave tiles (32 rows of one tree, a range's two trees in two tiles) and, up to 3,072 of
    them, its quad tiles of 8 rows."""
    seed, r = 4321 + n, _rand_u32(n, n)
    lo, hi = (1 << nbits) // 5, (1 << nbits) - 3
    kb = fss.KeyBatch(kind, nbits, n)
    for t in kb.key:
        t.fill_(0xA5)
    fss.fss_keygen(seed, 2, 5, lo, hi if kind else 0, T(r), kb)
    want = ofss.keygen_range(nbits, seed, 2, 5, lo, hi, r) if kind else ofss.keygen_eq(nbits, seed, 2, 5, lo, r)
    for b in range(2):
        got = from_device(kind, nbits, n, B(kb.key[b], kb.bytes_per_party))
        assert got.tobytes() == want[b].tobytes()


@pytest.mark.parametrize("n_edges", [1, 511, 513, 2049, 70001])
@pytest.mark.parametrize("npred", [(0, 0, 0), (1, 0, 2), (0, 3, 0), (2, 1, 1), (1, 1, 3), (0, 0, 4)])
def test_tail_tile_edges(fss, n_edges, npred):
    """One hop whose vertices and edge carry `npred` predicates, bits given: folds and the join at the edges
    of 16-word tiles, against the plan rebuilt from the oracle's triples."""
    seed, qid, nv = 5 + n_edges, 11, 700
    rng = np.random.default_rng(n_edges + 7 * sum(npred))
    src, dst = (rng.integers(0, nv, n_edges).astype(np.uint32) for _ in range(2))
    rows = (nv, nv, n_edges)
    preds, bits, and_id = [], [], 0
    for t in range(3):
        bits.append([])
        for _ in range(npred[t]):
            m = ofss.valid_mask(rows[t])
            b = [_rand_u32(int(rng.integers(1 << 30)), m.size) & m for _ in range(2)]
            bits[t].append(b)
            preds.append((t, None, None, (T(b[0]), T(b[1]))))
    plan = fss.Plan(seed, qid, 2, nv, n_edges, preds, T(src), T(dst)).allocate()
    fss.match_query(plan)

    def beaver(x, y, n):
        nonlocal and_id
        trip = ofss.triples(seed, qid, and_id, (n + 31) // 32)
        and_id += 1
        return ofss.beaver_and(x, y, trip, n)

    folds = []
    for t in range(3):
        acc = None
        for b in bits[t]:
            acc = b if acc is None else beaver(acc, b, rows[t])
        folds.append(acc)
    ends = [None if folds[t] is None else [ofss.pack_bits(ofss.unpack_bits(folds[t][b], nv)[ix]) for b in range(2)]
            for t, ix in ((0, src), (1, dst))]
    r = ends[0] if ends[1] is None else ends[1] if ends[0] is None else beaver(ends[0], ends[1], n_edges)
    if folds[2] is not None:
        r = folds[2] if r is None else beaver(r, folds[2], n_edges)
    if r is None:
        r = [ofss.valid_mask(n_edges), np.zeros((n_edges + 31) // 32, np.uint32)]
    for b in range(2):
        np.testing.assert_array_equal(U(plan.out[b]), r[b])
