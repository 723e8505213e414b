"""Prefix sums of one tile, of several and of more tiles than are added up directly: the
k = 1 lists of a path are its adjacency rows, at every offset."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 2047, 2048, 2049, 4097, 2048 * 2048, 2048 * 2048 + 1])
def test_row_offsets_of_a_path(n):
    require_gpu()
    from paper_1606_02162_amd import gila
    rp = np.minimum(np.maximum(2 * np.arange(n + 1, dtype=np.int64) - 1, 0), 2 * n - 2)
    ids = np.arange(n, dtype=np.int32)
    ci = np.stack([ids - 1, ids + 1], 1).ravel()[1:-1]
    g = inputs.Graph(n=n, row_ptr=rp, col_idx=np.ascontiguousarray(ci))
    kh = gila.build_khop(*gila.to_device_csr(g), 1)
    ptr, idx = kh.export()
    kh.free()
    assert np.array_equal(ptr, rp)
    assert np.array_equal(idx, ci)
