"""The device checks of a caller's CSR at their edges: tiles of 1024 entries,
rows that span tiles, and asymmetries that only the search in the shorter row
or only the count of unsearched entries can see."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    require_gpu()
    from paper_1606_02162_amd import gila
    return gila


def _status(G, rp, ci):
    import torch
    r = torch.tensor(np.asarray(rp), dtype=torch.int64, device="cuda")
    c = torch.tensor(np.asarray(ci), dtype=torch.int32, device="cuda")
    try:
        G.build_khop(r, c, 1).free()
    except G.GilaError as e:
        return str(e)
    return ""


BAD = {
    # every searched mirror is there; entries (0, 1) and (4, 1) have none
    "unsearched": ([0, 1, 3, 4, 5, 6], [1, 2, 3, 1, 1, 1], "not symmetric"),
    # equal rows: two directed triangles
    "cycles": ([0, 1, 2, 3, 4, 5, 6], [1, 2, 0, 4, 5, 3], "not symmetric"),
    "descending": ([0, 2, 3, 4], [2, 1, 0, 0], "not strictly ascending"),
    "loop": ([0, 1, 2], [0, 1], "self-loop"),
    "column": ([0, 1, 2], [1, 2], "column out of range"),
    "decreasing": ([0, 2, 1, 2], [1, 2], "row_ptr not monotone"),
    "past the end": ([0, 9, 1, 2], [1, 2], "row_ptr not monotone"),
    "first": ([1, 1, 2], [1, 0], "row_ptr[0] must be 0"),
    "odd": ([0, 1, 1], [1], "nnz must be even"),
}


@pytest.mark.parametrize("name", list(BAD))
def test_malformed(G, name):
    rp, ci, message = BAD[name]
    print(name, flush=True)
    assert message in _status(G, rp, ci)


@pytest.mark.parametrize("leaves", [1, 511, 512, 513, 1024, 5000])
def test_rows_across_tiles(G, leaves):
    """A star's hub row starts mid-tile and spans several; then one mirror is
    pointed elsewhere."""
    g = inputs.star_graph(leaves)
    print(g.name, flush=True)
    assert _status(G, g.row_ptr, g.col_idx) == ""
    if leaves > 2:
        ci = g.col_idx.copy()
        ci[-1] = 1  # the last leaf names the first one instead of the hub
        assert "not symmetric" in _status(G, g.row_ptr, ci)
