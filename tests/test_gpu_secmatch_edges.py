"""secMatch at the edges of its arguments: results equal the oracle's, share for share."""
import numpy as np
import pytest

import synth
from gpu_util import DEV
from oracle import secmatch as osm
from test_gpu_secmatch import K, PRF, SLOT_SEED, _gpu_graph, lib  # noqa: F401  (lib: the module's fixture)
from test_oracle_secmatch import DEGREES, DOMAINS, N, QUERIES

pytestmark = pytest.mark.gpu


def _equal(lib, q, seed, counter, seed0):  # noqa: F811
    fss, secmatch = lib
    tg = synth.typed_graph(seed, N, DOMAINS, DEGREES)
    shares = synth.typed_shares(seed, tg)
    want, _ = osm.sec_match(tg, osm.encode(tg, shares, K, SLOT_SEED + seed), q, 40 + seed, PRF, counter, seed0)
    got = secmatch.sec_match(_gpu_graph(lib, tg, shares, SLOT_SEED + seed), q, 40 + seed, PRF, counter, seed0, device=DEV)
    assert len(got) == len(want) > 0
    for gc, wc in zip(got, want):
        for gr, wr in zip(gc, wc):
            for j in range(3):
                np.testing.assert_array_equal(gr[j], wr[j])


@pytest.mark.parametrize("seed0", [2**62, 2**63 - 7, 2**63 + 5])
def test_any_64_bit_shuffle_seed(lib, seed0):  # noqa: F811
    _equal(lib, QUERIES[0], 1, 7, seed0)


@pytest.mark.parametrize("span,most", [(1, 1 << 20), (1 << 20, 1)])
def test_groups_in_several_library_calls(lib, monkeypatch, span, most):  # noqa: F811
    """Groups whose rows one call does not number (here a lowered limit) go in several calls with the same results."""
    fss, secmatch = lib
    monkeypatch.setattr(secmatch, "ROW_SPAN", span)
    monkeypatch.setattr(secmatch, "CALL_ROWS", most)
    calls = []
    one = fss.rss_sec_fetch_groups
    monkeypatch.setattr(fss, "rss_sec_fetch_groups", lambda src, *a, **k: calls.append(src.size) or one(src, *a, **k))
    _equal(lib, QUERIES[0], 1, 7, 600)
    assert len(calls) > len(QUERIES[0].targets)
