"""Batches that are accepted on the host whatever their number of tiles."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as f
    return f


@pytest.mark.parametrize("kind", ["EQ", "RANGE"])
def test_eval_batch_of_more_tiles_than_32_bits(fss, kind):
    """1,100 requests of 2^28 rows (2^36 rows and more): no longer refused for their number.  Without a queue the
    call ends at its workspace check, after the count of tiles and before any launch."""
    kb = fss.fss_keybatch(getattr(fss, kind), 32, (1 << 28) - 1, (ctypes.c_void_p * 2)(256, 512))
    reqs = (fss.fss_eval_req * 1100)(*[fss.fss_eval_req(0, 0, ctypes.pointer(kb), 4096, 4096)] * 1100)
    assert fss.LIB.fss_eval_batch(reqs, 1100, None, 0, None) == fss.ENOMEM
