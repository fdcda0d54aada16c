"""Host parts of secMatch that need no GPU."""
import numpy as np
import pytest

from paper_2209_03526_amd import secmatch


@pytest.mark.parametrize("base", [0, 5, 2**62, 2**63 - 4, 2**63 + 5, 2**64 - 1, 2**64 + 7, -3])
def test_seeds_of_any_64_bits(base):
    """Every 64-bit seed (and what wraps past it) gives the low 64 bits of base + step."""
    steps = np.array([0, 1, 2, 3, 3_000_000_001], np.int64)
    assert secmatch._plus(base, steps) == [(base + int(v)) % 2**64 for v in steps]
