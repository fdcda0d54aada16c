"""rss_sec_access_batch beyond independent calls over short lists: calls that
read an earlier call's outputs, against the same calls made one by one, and
lists of one length, records of more than a tile, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, T, U
from oracle import access

pytestmark = pytest.mark.gpu

KEYS = (51, 52, 53)


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as f
    return f


def _words(rng, n):
    return T(rng.integers(0, 2**32, max(1, n), dtype=np.uint64).astype(np.uint32))


class _Lists:
    """Posting lists of random words over `ids` IDs, and a batch's output buffers and arguments."""

    def __init__(self, fss, rng, lens, ids, calls, attr_words=2):
        self.fss, self.n, self.ids, self.calls, self.wd = fss, lens.size, ids, calls, attr_words
        self.wx, self.lmax = (ids + 31) // 32, int(lens.max())
        self.d_off = T(np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32))
        self.post = [_words(rng, int(lens.sum()) * self.wx) for _ in range(3)]
        self.attr = [_words(rng, ids * attr_words) for _ in range(3)]
        self.idm = [[_words(rng, (self.n + 31) // 32) for _ in range(3)] for _ in range(calls)]
        self.counters = [7 + 2 * c for c in range(calls)]
        self.seeds = [int(v) for v in rng.integers(0, 2**62, 3 * calls)]

    def outputs(self):
        full = lambda k: torch.full((k,), -1, dtype=torch.int32, device=DEV)  # noqa: E731
        m, t, a = self.calls, self.lmax * self.wx, self.lmax * self.wd
        return [full(m * t) for _ in range(3)], [full(m * a) for _ in range(3)], full(m * self.lmax), full(m)

    def batch(self, out, ptrs):
        self.fss.rss_sec_access_batch(self.n, self.ids, ptrs, self.d_off, self.lmax, self.post, self.wd, self.attr, KEYS,
                                      self.counters, self.seeds, *out)

    def singles(self, out, idm):
        """Call c reads idm(c) (three tensors, taken when its turn comes)."""
        ids, attrs, rows, count = out
        t, a = self.lmax * self.wx, self.lmax * self.wd
        for c in range(self.calls):
            self.fss.rss_sec_access(self.n, self.ids, idm(c), self.d_off, self.lmax, self.post, self.wd, self.attr, KEYS,
                                    self.counters[c], self.seeds[3 * c:3 * c + 3], [x[c * t:(c + 1) * t] for x in ids],
                                    [x[c * a:(c + 1) * a] for x in attrs], rows[c * self.lmax:(c + 1) * self.lmax],
                                    count[c:c + 1])


def _equal(got, want):
    for g, w in zip(list(got[0]) + list(got[1]) + list(got[2:]), list(want[0]) + list(want[1]) + list(want[2:])):
        np.testing.assert_array_equal(U(g), U(w))


@pytest.mark.parametrize("reads", [{1: (0, 0)}, {1: (0, 1), 2: (1, 0), 4: (1, 2)}, {5: (4, 3)}, {9: (0, 0), 3: (2, 5)}])
def test_calls_that_read_an_earlier_calls_ids(fss, reads):
    """Candidates and neighbours of one type: call c's matched ID is row r of the IDs that call b < c keeps."""
    rng = np.random.default_rng(len(reads) + 40)
    n = 200
    L = _Lists(fss, rng, rng.integers(1, 9, n), n, 10)

    def idm(out):
        def of(c):
            if c not in reads:
                return L.idm[c]
            b, r = reads[c]
            at = (b * L.lmax + r) * L.wx
            return [x[at:at + L.wx] for x in out[0]]
        return of

    want = L.outputs()
    L.singles(want, idm(want))
    got = L.outputs()
    L.batch(got, [t.data_ptr() for c in range(L.calls) for t in idm(got)(c)])
    _equal(got, want)


@pytest.mark.parametrize("n,length,ids,calls", [(700, 12, 9000, 8), (700, 12, 9000, 4), (2100, 24, 100, 8), (90, 40, 321, 2),
                                                (1, 5, 33, 5), (65, 1, 64, 9), (300, 9, 20, 1), (2100, 24, 100, 1),
                                                (300, 7, 4096, 1), (300, 7, 4097, 1)])
def test_equal_lists_and_wide_records_equal_oracle(fss, n, length, ids, calls):
    """Lists of one length (every slot as full as the first), records of one word to more than a tile of 256 words,
    four and eight calls a pass: kept IDs, attributes and counts equal the oracle's single calls."""
    rng = np.random.default_rng(n + ids)
    L = _Lists(fss, rng, np.full(n, length), ids, calls)
    out = L.outputs()
    L.batch(out, [t.data_ptr() for c in L.idm for t in c])
    post = [U(t).reshape(-1, L.wx) for t in L.post]
    attr = [U(t).reshape(ids, L.wd) for t in L.attr]
    bits = lambda t: np.unpackbits(U(t).view(np.uint8), bitorder="little")[:n]  # noqa: E731
    for c in range(0, calls, 3):
        want_ids, want_attrs = access.sec_access_csr([bits(t) for t in L.idm[c]], post, np.arange(n + 1) * length, attr, ids,
                                                     list(KEYS), L.seeds[3 * c:3 * c + 3], L.counters[c])
        m = want_ids[0].shape[0]
        assert U(out[3])[c] == m
        for i in range(3):
            np.testing.assert_array_equal(U(out[0][i]).reshape(calls, length, L.wx)[c, :m], want_ids[i])
            np.testing.assert_array_equal(U(out[1][i]).reshape(calls, length, L.wd)[c, :m], want_attrs[i])


@pytest.mark.parametrize("length,ids,calls", [(2, 40, 2), (15, 40, 2), (16, 40, 2), (17, 40, 3), (511, 40, 2), (512, 40, 2),
                                              (513, 40, 3), (1023, 33, 2), (1024, 33, 2)])
def test_shuffles_side_by_side_at_the_rankings_edges(fss, length, ids, calls):
    """Fetched lists that a workgroup each shuffles: rows ranked by several threads, by one, odd numbers of rows."""
    test_equal_lists_and_wide_records_equal_oracle(fss, 3, length, ids, calls)
