"""Rows about the longest that one wavefront builds, and about its sort's sizes: bit-exact
against the oracle's BFS, and the same lists as every row by a whole workgroup."""
import numpy as np
import pytest

from gpu_common import oracle_rows, require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


def _graph(kind):
    """Disjoint cliques, stars or paths whose k-hop rows have 1, 63 .. 65, 127 .. 129,
    255 .. 257 and 510 .. 515 ids, ids shuffled."""
    sizes = (2, 3, 64, 65, 66, 128, 129, 130, 256, 257, 258, 511, 512, 513, 514, 516)
    edges, base = [], 0
    for size in sizes:
        if kind == "clique":
            i, j = np.triu_indices(size, 1)
        elif kind == "star":
            i, j = np.zeros(size - 1, np.int64), np.arange(1, size)
        else:  # two hubs joined by an edge: a row of both at k = 2, of each at k = 1
            i = np.r_[np.zeros(size // 2, np.int64), np.full(size - size // 2 - 1, size // 2), 0]
            j = np.r_[np.arange(1, size // 2 + 1), np.arange(size // 2 + 1, size), size // 2]
        edges.append(np.stack([i + base, j + base], 1))
        base += size
    u, v = np.concatenate(edges).T
    base += 7  # isolated vertices
    p = np.random.default_rng(3).permutation(base)
    return inputs.to_csr(base, p[u], p[v], kind)


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("kind", ["clique", "star", "hubs"])
def test_rows_about_the_cap(kind, k, monkeypatch):
    require_gpu()
    from paper_1606_02162_amd import gila
    g = _graph(kind)
    rp, ci = gila.to_device_csr(g)
    optr, oidx = oracle_rows(g, k)
    orders = []
    for bitmap in (None, "lds"):
        if bitmap:
            monkeypatch.setenv("GILA_BFS_BITMAP", bitmap)
        kh = gila.build_khop(rp, ci, k)
        ptr, idx = kh.export()
        orders.append(kh.order())
        kh.free()
        assert np.array_equal(ptr, optr), (kind, k, bitmap)
        assert np.array_equal(idx, oidx), (kind, k, bitmap)
    assert np.array_equal(orders[0], orders[1])
