"""Host parts of secMatch that need no GPU."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2209_03526_amd import secmatch


@pytest.mark.parametrize("base", [0, 5, 2**62, 2**63 - 4, 2**63 + 5, 2**64 - 1, 2**64 + 7, -3])
def test_seeds_of_any_64_bits(base):
    """Every 64-bit seed (and what wraps past it) gives the low 64 bits of base + step."""
    steps = np.array([0, 1, 2, 3, 3_000_000_001], np.int64)
    assert secmatch._plus(base, steps) == [(base + int(v)) % 2**64 for v in steps]


@pytest.mark.parametrize("whole", [0, 1 << 18])
def test_results_copy_the_kept_records_alone(monkeypatch, whole):
    """Two targets of 500 and 3 x 40 candidates, few of them kept: the results are the kept vertices' ID words,
    group by group, and no more than those leave the device (small buffers are copied whole)."""
    monkeypatch.setattr(secmatch, "WHOLE_COPY", whole, raising=False)
    rng = np.random.default_rng(1)
    n, domain = {"U": 500, "P": 100}, {("U", "a"): 40, ("P", "b"): 70}
    graph = SimpleNamespace(n=n, domains=domain)
    query = SimpleNamespace(targets=[SimpleNamespace(vtype="U", attr="a"), SimpleNamespace(vtype="P", attr="b")],
                            parent=lambda i: i - 1)
    targets, plain = [], []
    for t, name, sizes, nkept, parent in (("U", "a", [500], [2], [None]), ("P", "b", [40, 40, 40], [1, 0, 3], [(0, 0), (0, 1), (0, 1)])):
        wi, wv = secmatch.words(n[t]), secmatch.words(domain[(t, name)])
        kept = [rng.integers(-2**31, 2**31, (sum(sizes), wi + wv), dtype=np.int64).astype(np.int32) for _ in range(3)]
        row0 = np.cumsum(sizes) - sizes
        targets.append(secmatch._Target(None, None, None, np.array(sizes), parent, torch.from_numpy(np.stack(kept)),
                                        row0, np.array(nkept)))
        plain.append([[[k[row0[g] + r, :wi].view(np.uint32) for k in kept] for r in range(nkept[g])] for g in range(len(sizes))])
    want = [[plain[0][0][0], plain[1][0][0]]] + [[plain[0][0][1], plain[1][2][r]] for r in range(3)]
    moved, cpu = [], torch.Tensor.cpu
    monkeypatch.setattr(torch.Tensor, "cpu", lambda self, *a, **k: moved.append(self.numel()) or cpu(self, *a, **k))
    got = secmatch._results(targets, query, graph)
    assert len(got) == len(want)
    for g, w in zip(got, want):
        for gr, wr in zip(g, w):
            for j in range(3):
                np.testing.assert_array_equal(gr[j], wr[j])
    assert whole or sum(moved) <= 3 * (2 * secmatch.words(500) + 4 * secmatch.words(100))


@pytest.mark.parametrize("span,most", [(1 << 32, (1 << 31) - 1), (100, 1000), (1 << 20, 33), (1, 1)])
def test_row_runs(monkeypatch, span, most):
    """Runs of groups that one library call numbers: every group once, in order, within the span and the rows a call
    takes (unless it is alone); one run where all fit."""
    monkeypatch.setattr(secmatch, "ROW_SPAN", span)
    monkeypatch.setattr(secmatch, "CALL_ROWS", most)
    rng = np.random.default_rng(5)
    n = rng.integers(1, 24, 50)
    base = np.arange(50) * 24
    runs = secmatch._row_runs(base, n)
    assert [g for lo, hi in runs for g in range(lo, hi)] == list(range(50))
    for lo, hi in runs:
        assert hi - lo == 1 or (base[hi - 1] + n[hi - 1] - base[lo] <= span and n[lo:hi].sum() <= most)
        if hi < 50:
            assert base[hi] + n[hi] - base[lo] > span or n[lo:hi + 1].sum() > most
    assert span < 1 << 20 or most < 1000 or len(runs) == 1


def test_row_numbers_past_32_bits():
    """2^22 calls' lists of 1,024: the rows of the last groups lie past 2^32, in a second run."""
    base = np.arange((1 << 22) + 3) * 1024
    live = np.array([0, 1, (1 << 22) - 1, 1 << 22, (1 << 22) + 2])
    runs = secmatch._row_runs(base[live], np.full(5, 7))
    assert runs == [(0, 3), (3, 5)]
