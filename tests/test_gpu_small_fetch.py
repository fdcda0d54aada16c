"""Shuffles and fetches around the line between one workgroup and launches over
the chip (64 rows; 128 rows and 256 slices, a fetch's 320), against the oracle."""
import pytest

import test_gpu_compact
from test_gpu_compact import fss  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w", [(96, 16), (128, 32), (128, 33), (129, 16), (85, 48), (86, 48), (65, 63), (64, 255), (126, 7),
                                 (106, 48), (107, 48)])
def test_at_the_line(fss, n, w):  # noqa: F811
    test_gpu_compact.test_small_shuffles_and_fetches(fss, n, w)

