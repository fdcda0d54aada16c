"""Sizes that secAccess refuses on the host, before anything is enqueued."""
import ctypes

import pytest
import torch


@pytest.fixture(scope="module")
def fss():
    from paper_2209_03526_amd import fss as f
    return f


@pytest.mark.parametrize("x_bits,attr_words", [(1 << 31, 1), (32, 1 << 31)])
def test_fetched_records_past_the_prfs_blocks(fss, x_bits, attr_words):
    """More than 2^36 words of fetched IDs or attributes would repeat PRF blocks: refused, as the re-share refuses them."""
    if torch.cuda.is_available():
        pytest.skip("made-up addresses")
    P, u64 = ctypes.c_void_p, ctypes.c_uint64
    p = P(4096)
    three = (P * 3)(4096, 4096, 4096)
    keys = (u64 * 3)(1, 2, 3)
    assert fss.LIB.rss_sec_access(64, x_bits, three, p, 65535, three, attr_words, three, keys, 1, keys, three, three, p, p, p,
                                  1 << 62, None) == fss.EUNSUPPORTED
    assert b"2^36" in fss.LIB.fss_last_error()
