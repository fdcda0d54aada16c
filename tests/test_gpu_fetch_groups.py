"""rss_sec_fetch_groups against the calls that it stands for, group by group
(rss_sec_eval_records, rss_reshare, rss_fetch_table, rss_fetch_many, each pinned
to the oracle elsewhere): groups of no, one and many rows, more than one launch
of them, and groups too large for one workgroup's shuffle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, T, U

pytestmark = pytest.mark.gpu

KEYS, COUNTER = (51, 52, 53), 9


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as lib
    return lib


CASES = [([1], 40, 7), ([0, 3, 0, 32, 33], 100, 0), ([1024, 5], 17, 14), ([1025, 2, 0, 700], 64, 5),
         ([1 + i % 3 for i in range(70)], 100, 31), ([40] * 65, 33, 3), ([300], 100, 250)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_fetch_groups_equal_the_single_calls(fss, case):
    n, npos, wi = CASES[case]
    rng = np.random.default_rng(case)
    n = np.array(n, np.uint32)
    wv = (npos + 31) // 32
    rec, gap = wi + wv, 3
    src = (np.cumsum(n + gap) - n).astype(np.uint32)             # groups apart from one another
    rows = int(src[-1] + n[-1])
    words = lambda k: T(rng.integers(0, 2**32, max(1, k), dtype=np.uint64).astype(np.uint32))  # noqa: E731
    evals = [words(wv) for _ in range(6)]
    ids, vals = [words(rows * wi) for _ in range(3)], [words(rows * wv) for _ in range(3)]
    seeds = [int(v) for v in rng.integers(0, 2**62, 3 * n.size)]
    total = int(n.sum())
    full = lambda k: torch.full((max(1, k),), -1, dtype=torch.int32, device=DEV)  # noqa: E731
    out, pos, cnt = [full(total * rec) for _ in range(3)], full(total), full(n.size)
    fss.rss_sec_fetch_groups(src, n, npos, evals, wi, ids if wi else [None] * 3, vals, KEYS, COUNTER, seeds, out, pos, cnt)
    row = 0
    for g, (s, k) in enumerate(zip(src.tolist(), n.tolist())):
        if k == 0:
            assert U(cnt)[g] == 0
            continue
        gi, gv = [t[s * wi:(s + k) * wi] for t in ids], [t[s * wv:(s + k) * wv].contiguous() for t in vals]
        x3, z3 = [full((k + 31) // 32) for _ in range(3)], [full((k + 31) // 32) for _ in range(3)]
        for i in range(3):
            fss.rss_sec_eval_records(k, npos, evals[2 * i], evals[2 * i + 1], gv[i], gv[(i + 1) % 3], x3[i])
        fss.rss_reshare(k, x3, KEYS, COUNTER + g, z3)
        table, kept = [full(k * (1 + rec)) for _ in range(3)], [full(k * rec) for _ in range(3)]
        fss.rss_fetch_table(k, z3, wi, gi if wi else None, wv, gv, table)
        p1, c1 = full(k), full(1)
        fss.rss_fetch_many(k, 1 + rec, table, seeds[3 * g:3 * g + 3], kept, p1, c1)
        m = int(U(c1)[0])
        assert U(cnt)[g] == m
        np.testing.assert_array_equal(U(pos)[row:row + m], U(p1)[:m])
        for i in range(3):
            np.testing.assert_array_equal(U(out[i])[row * rec:(row + m) * rec], U(kept[i])[:m * rec])
        row += k
