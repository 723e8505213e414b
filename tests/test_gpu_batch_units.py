"""k-hop lists of a batch whose graphs take several units of sources each, and whose
frontiers do and do not fit the wavefront's list: bit-exact against the oracle's BFS."""
import numpy as np
import pytest

from gpu_common import oracle_rows, require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 5])
def test_units_and_frontier_lists(k):
    require_gpu()
    from paper_1606_02162_amd import gila
    # one source more and less than a unit; levels of 1200 new ids under a list of 128 to
    # 150 entries (stars, a hub of stars) and levels of a handful
    u, v = [], []
    for i in range(1, 41):
        u += [0] + [i] * 30
        v += [i] + list(range(41 + 30 * (i - 1), 41 + 30 * i))
    graphs = [inputs.path_graph(511), inputs.path_graph(512), inputs.path_graph(513),
              inputs.star_graph(1200), inputs.to_csr(41 + 1200, u, v, "hub of stars"),
              inputs.grid_graph(33, 33), inputs.barabasi_albert(1500, 3, 7),
              inputs.random_tree_plus_edges(2400, 300, 9), inputs.path_graph(1),
              inputs.complete_graph(150)]
    b = gila.Batch([gila.to_device_csr(g) for g in graphs], [k] * len(graphs))
    for i, g in enumerate(graphs):
        ptr, idx = b.export(i, g.n)
        optr, oidx = oracle_rows(g, k)
        assert np.array_equal(ptr, optr), (g.name, k)
        assert np.array_equal(idx, oidx), (g.name, k)
    b.free()


@pytest.mark.parametrize("k", [1, 2, 3, 5])
@pytest.mark.parametrize("largest", [100, 279, 280, 281, 283, 284, 285])
def test_graphs_that_just_fit_in_lds(k, largest):
    """Beside a complete graph that just fits (the LDS of a workgroup then holds lists of 18 ids
    instead of 128): levels of one id, of a few and of nearly all; bit-exact again."""
    require_gpu()
    from paper_1606_02162_amd import gila
    print(f"batch lds {largest} k={k}", flush=True)
    graphs = [inputs.complete_graph(largest), inputs.star_graph(90), inputs.path_graph(99),
              inputs.grid_graph(9, 10), inputs.barabasi_albert(95, 3, 2), inputs.path_graph(2)]
    b = gila.Batch([gila.to_device_csr(g) for g in graphs], [k] * len(graphs))
    for i, g in enumerate(graphs):
        ptr, idx = b.export(i, g.n)
        optr, oidx = oracle_rows(g, k)
        assert np.array_equal(ptr, optr), (g.name, k)
        assert np.array_equal(idx, oidx), (g.name, k)
    b.free()
