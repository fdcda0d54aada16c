"""Plan tails in 64-word tiles at ragged sizes: joins of more than 2^23 edges and
folds of more than 2^21 rows (below, the tiles have 16 words), bits given,
against the plan rebuilt from the oracle's triples."""
import numpy as np
import pytest
import torch

from gpu_util import T, U
from oracle import fss as ofss
import test_gpu_tiles
from test_gpu_tiles import fss  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_edges,npred", [((1 << 23) + 33, (1, 1, 3)), ((1 << 23) + 2049, (2, 0, 1)), ((1 << 23) + 70001, (0, 0, 4)),
                                           (1 << 23, (1, 2, 1))])
def test_joins(fss, n_edges, npred):  # noqa: F811
    test_gpu_tiles.test_tail_tile_edges(fss, n_edges, npred)


@pytest.mark.parametrize("n", [(1 << 21) + 1, (1 << 21) + 2049, (1 << 21) + 70001, 1 << 21])
@pytest.mark.parametrize("hop", [False, True])
def test_folds(fss, n, hop):  # noqa: F811
    """Three predicates on one vertex table: the output of a one-vertex query, or the pairs that a join gathers
    (the first and the last 2,000 rows)."""
    seed, qid, rng = n, 3, np.random.default_rng(n)
    mask = ofss.valid_mask(n)
    bits = [[rng.integers(0, 2**32, mask.size, dtype=np.uint64).astype(np.uint32) & mask for _ in range(2)] for _ in range(3)]
    preds = [(0, None, None, (T(b[0]), T(b[1]))) for b in bits]
    fold = bits[0]
    for k in (1, 2):
        fold = ofss.beaver_and(fold, bits[k], ofss.triples(seed, qid, k - 1, mask.size), n)
    if not hop:
        plan = fss.Plan(seed, qid, 1, n, 0, preds).allocate()
        want = fold
    else:
        src = np.concatenate([np.arange(2000), n - 1 - np.arange(2000)]).astype(np.uint32)
        dst = np.zeros(4000, np.uint32)
        plan = fss.Plan(seed, qid, 2, n, 4000, preds, T(src), T(dst)).allocate()
        want = [ofss.pack_bits(ofss.unpack_bits(f, n)[src]) for f in fold]
    fss.match_query(plan)
    torch.cuda.synchronize()
    for b in range(2):
        np.testing.assert_array_equal(U(plan.out[b], want[b].size), want[b])
