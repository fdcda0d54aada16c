"""The compaction of tables of few, wide records, whose blocks several
workgroups copy: kept records, positions and count as for narrow ones."""
import pytest

import test_gpu_compact
from test_gpu_compact import fss  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [False, True])
@pytest.mark.parametrize("parity", [False, True])
@pytest.mark.parametrize("n,w,share", [(70, 2000, 0.5), (300, 501, 1.0), (1025, 257, 0.02), (2000, 500, 0.5), (8000, 256, 0.9)])
def test_kept_wide_records(fss, n, w, share, parity, off):  # noqa: F811
    test_gpu_compact.test_kept_records(fss, n, w, share, parity, off)
