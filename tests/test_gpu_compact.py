"""The multi-workgroup compaction of secFetch and of the secAccess filter, and
the permutations' small chunks, at their edges: kept records, positions and
count against the shuffled shares that rss_shuffle gives for the same seeds."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, T, T_off, U, empty_off
from oracle import shuffle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as lib
    return lib


@pytest.mark.parametrize("off", [False, True])
@pytest.mark.parametrize("parity", [False, True])
@pytest.mark.parametrize("n,w,share", [(1025, 16, 0.5), (1279, 2, 1.0), (2049, 5, 0.0), (65536, 7, 0.01), (262144, 4, 0.5),
                                       (262145, 3, 0.9), (524289, 17, 0.3), (1100, 70, 0.5)])
def test_kept_records(fss, n, w, share, parity, off):
    rng = np.random.default_rng(n + w)
    u32 = lambda *k: rng.integers(0, 2**32, k, dtype=np.uint64).astype(np.uint32)  # noqa: E731
    sh = [u32(n, w) for _ in range(3)]
    keep = rng.random(n) < share                         # bit 0 of word 0, or the parity of the record
    opened = sh[0] ^ sh[1] ^ sh[2]
    now = np.bitwise_count(opened).sum(axis=1) & 1 if parity else opened[:, 0] & 1
    sh[2][:, 0] ^= (now != keep).astype(np.uint32)
    seeds = [11 + n, 12, 13]
    put, buf = (T_off, empty_off) if off else (T, lambda k: torch.empty(k, dtype=torch.int32, device=DEV))
    dev = [put(s.ravel()) for s in sh]
    out = [buf(n * w) for _ in range(3)]
    fss.rss_shuffle(n, w, dev, seeds, out)
    want = [U(o).reshape(n, w) for o in out]
    plain = want[0] ^ want[1] ^ want[2]
    rows = np.flatnonzero(np.bitwise_count(plain).sum(axis=1) & 1 if parity else plain[:, 0] & 1)
    assert rows.size == keep.sum()
    rw = w if parity else w - 1
    kept, pos, cnt = [buf(n * rw) for _ in range(3)], buf(n), buf(1)
    for t in kept + [pos]:
        t.fill_(-1)
    (fss.rss_compact_valid if parity else fss.rss_fetch_many)(n, w, dev, seeds, kept, pos, cnt)
    assert U(cnt)[0] == rows.size
    np.testing.assert_array_equal(U(pos)[:rows.size], rows)
    assert (U(pos)[rows.size:] == 0xFFFFFFFF).all()
    for i in range(3):
        got = U(kept[i])
        np.testing.assert_array_equal(got[:rows.size * rw].reshape(-1, rw), want[i][rows][:, w - rw:])
        assert (got[rows.size * rw:] == 0xFFFFFFFF).all()


@pytest.mark.parametrize("n,w", [(1, 3), (64, 16), (65, 16), (64, 300), (127, 5), (128, 16), (129, 4), (255, 17), (513, 2),
                                 (1023, 16), (1024, 33)])
def test_small_shuffles_and_fetches(fss, n, w):
    """Tables that one workgroup shuffles (up to 64 rows) and those that several rank, 128 rows each."""
    rng = np.random.default_rng(n * w)
    sh = [rng.integers(0, 2**32, (n, w), dtype=np.uint64).astype(np.uint32) for _ in range(3)]
    seeds = (31 + n, 32 + w, 33)
    dev, out = [T(s.ravel()) for s in sh], [torch.empty(n * w, dtype=torch.int32, device=DEV) for _ in range(3)]
    fss.rss_shuffle(n, w, dev, seeds, out)
    want = shuffle.sec_shuffle(sh, *seeds)
    for i in range(3):
        np.testing.assert_array_equal(U(out[i]).reshape(n, w), want[i])
    for parity in (False, True):
        plain = want[0] ^ want[1] ^ want[2]
        rows = np.flatnonzero(np.bitwise_count(plain).sum(axis=1) & 1 if parity else plain[:, 0] & 1)
        rw = w if parity else w - 1
        kept, pos, cnt = [torch.empty(n * rw, dtype=torch.int32, device=DEV) for _ in range(3)], T(np.zeros(n)), T([0])
        (fss.rss_compact_valid if parity else fss.rss_fetch_many)(n, w, dev, seeds, kept, pos, cnt)
        assert U(cnt)[0] == rows.size
        np.testing.assert_array_equal(U(pos)[:rows.size], rows)
        for i in range(3):
            np.testing.assert_array_equal(U(kept[i])[:rows.size * rw].reshape(-1, rw), want[i][rows][:, w - rw:])


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4097, 131073, 262144, 262145])
def test_permutations_at_chunk_edges(fss, n):
    seeds = [1000 + n, 2000 + n, 3000 + n]
    perms = torch.empty(3 * n, dtype=torch.int32, device=DEV)
    fss.rss_shuffle_prepare(n, seeds, perms)
    got = U(perms).reshape(3, n)
    for k, (seed, p, inverse) in enumerate(((seeds[0], 0, True), (seeds[2], 2, True), (seeds[1], 1, False))):
        want = shuffle.permutation(seed, p, n)
        if inverse:
            want = np.argsort(want)
        np.testing.assert_array_equal(got[k], want)
