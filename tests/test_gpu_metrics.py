"""GPU parity of the drawing-quality metrics (Section 5.2) against the
oracle: crossings (total and per edge) and per-vertex Jaccard indices
bit-exact, edge length mean and deviation to 1e-12.  Degenerate drawings
(grid points: collinear and cocircular; coincident points; collinear points;
coordinates of very different magnitude, where rounded differences get the
orientation or in-disc sign wrong) are included, and the total without
per-edge counts (each pair tested once) must equal the total with them.
The Gabriel degrees are checked on both of the kernel's paths (a thread per
point, and a wavefront per point for searches over the thread's budget).
At full size (R-MAT 18): sampled per-edge crossings from the oracle, the
edge lengths in full, and the similarity against a Gabriel graph built
independently from scipy's Delaunay triangulation (a Delaunay edge is a
Gabriel edge when both angles opposite it are acute).
"""
import math
import os

import numpy as np
import pytest

import oracle
from gpu_common import require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    require_gpu()
    from paper_1606_02162_amd import gila
    return gila


def _grid_xy(rows, cols):
    n = rows * cols
    return np.stack([np.arange(n) % cols, np.arange(n) // cols], axis=1).astype(float) * 3.0


def metric_suite():
    out = []
    k = inputs.complete_graph(12)
    th = 0.3 + 2 * math.pi * np.arange(12) / 12
    out.append(("k12_convex", k, np.stack([100 * np.cos(th), 100 * np.sin(th)], 1)))
    g = inputs.grid_graph(12, 15)
    out.append(("grid_as_grid", g, _grid_xy(12, 15)))
    out.append(("grid_random", g, inputs.uniform_positions(g.n, seed=3, width=50.0)))
    e = inputs.erdos_renyi(400, 900, seed=5)
    out.append(("er400", e, inputs.uniform_positions(e.n, seed=6, width=500.0)))
    t = inputs.random_tree_plus_edges(500, 100, seed=7)
    x = inputs.uniform_positions(t.n, seed=8, width=300.0)
    x[10] = x[11]          # coincident points
    x[20] = x[21] = x[22]
    out.append(("tree_coincident", t, x))
    p = inputs.path_graph(60)
    out.append(("path_on_a_line", p, np.stack([np.arange(60.0) ** 1.5, np.zeros(60)], 1)))
    s = inputs.star_graph(40)
    out.append(("star", s, inputs.uniform_positions(s.n, seed=9, width=10.0)))
    # rounded differences get these signs wrong (the oracle's exact-sign pins)
    d1, d2 = float(np.float32(1e-20)), float(np.float32(2e-20))
    x = np.array([[d1, d2], [512.0, 512.0], [256.0, 256.0], [0.0, 512.0]])
    out.append(("tiny_crossing", inputs.to_csr(4, [0, 2], [1, 3]), x))
    out.append(("tiny_disc", inputs.path_graph(3), np.array([[d1, 0.0], [2.0, 0.0], [1.0, 1.0]])))
    rng = np.random.default_rng(5)
    vals = np.float32([0.0, 1e-20, -3e-20, 1.0, 2.0, 3.0, 1e-7, 1024.0, 1024.0000001, 5e9])
    for seed in (11, 12, 13):
        e = inputs.erdos_renyi(60, 300, seed=seed)
        out.append((f"near_degenerate{seed}", e, vals[rng.integers(0, vals.size, (60, 2))].astype(float)))
    return out


def _run(G, g, x, prec, what=7, per_edge=True):
    import torch
    rp, ci = G.to_device_csr(g)
    pos = torch.from_numpy(x).to(dtype=G.position_dtype(prec), device="cuda").contiguous()
    m = int(oracle.edge_list(g.row_ptr, g.col_idx).shape[0])
    ec = torch.full((max(m, 1),), -7, dtype=torch.int64, device="cuda")
    jac = torch.zeros(max(g.n, 1), dtype=torch.float64, device="cuda")
    out = G.drawing_metrics(rp, ci, prec, pos, what, ec if per_edge else None, jac)
    return out, ec.cpu().numpy()[:m], jac.cpu().numpy()[: g.n]


@pytest.fixture
def gabriel_budget(request):
    """GILA_GABRIEL_BUDGET for the test: None (the library's default), "0"
    (every point's Gabriel search on a wavefront of its own) or a small
    budget (a mix of both paths)."""
    old = os.environ.get("GILA_GABRIEL_BUDGET")
    if request.param is not None:
        os.environ["GILA_GABRIEL_BUDGET"] = request.param
    yield request.param
    if old is None:
        os.environ.pop("GILA_GABRIEL_BUDGET", None)
    else:
        os.environ["GILA_GABRIEL_BUDGET"] = old


@pytest.mark.parametrize("gabriel_budget", [None, "0", "40"], indirect=True)
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_metrics_small(G, precision, gabriel_budget):
    prec = G.PRECISIONS[precision]
    for name, g, x in metric_suite():
        print(f"metrics {name} {precision} budget {gabriel_budget}", flush=True)
        xs = oracle.single(x)
        out, ec, jac = _run(G, g, xs, prec)
        tot, per = oracle.crossings(g.n, g.row_ptr, g.col_idx, xs, per_edge=True)
        assert out.crossings == tot and np.array_equal(ec, per), name
        # without per-edge counts each pair is tested once
        once, _, _ = _run(G, g, xs, prec, what=G.METRIC_CROSSINGS, per_edge=False)
        assert once.crossings == tot, name
        mu, sd = oracle.edge_lengths(g.n, g.row_ptr, g.col_idx, xs)
        assert out.edge_length_mean == pytest.approx(mu, rel=1e-12, abs=1e-300)
        assert out.edge_length_std == pytest.approx(sd, rel=1e-10, abs=1e-12 * max(mu, 1.0))
        sim, pj = oracle.similarity(g.n, g.row_ptr, g.col_idx, xs, per_vertex=True)
        assert np.array_equal(jac, pj), name
        assert out.similarity == pytest.approx(sim, rel=1e-12)
        gp, _ = oracle.gabriel(xs)
        assert out.gabriel_edges == int(gp[-1]) // 2
        assert out.edges == g.m


def test_metric_flags_and_empty(G):
    import torch
    g = inputs.erdos_renyi(100, 200, seed=2)
    x = oracle.single(inputs.uniform_positions(g.n, seed=1, width=100.0))
    out, _, _ = _run(G, g, x, G.FP32, what=G.METRIC_LENGTHS)
    assert out.crossings == 0 and out.similarity == 1.0 and out.edge_length_mean > 0
    e = inputs.to_csr(5, [], [])
    out, _, jac = _run(G, e, oracle.single(inputs.uniform_positions(5, 2, 10.0)), G.FP32)
    assert out.edges == 0 and out.crossings == 0
    assert out.gabriel_edges > 0 and np.all(jac == 0.0)  # no graph edges, some Gabriel ones
    bad = torch.full((4, 2), float("nan"), device="cuda")
    rp, ci = G.to_device_csr(inputs.path_graph(4))
    with pytest.raises(G.GilaError) as err:
        G.drawing_metrics(rp, ci, G.FP32, bad, G.METRIC_SIMILARITY)
    assert err.value.code == G.GILA_EINVAL


def _delaunay_gabriel(x):
    """Gabriel edges as the Delaunay edges whose opposite angles are acute."""
    from scipy.spatial import Delaunay
    tri = Delaunay(x)
    opp = {}
    for s in tri.simplices:
        for a, b, c in ((s[0], s[1], s[2]), (s[1], s[2], s[0]), (s[2], s[0], s[1])):
            key = (min(a, b), max(a, b))
            opp.setdefault(key, []).append(c)
    adj = [[] for _ in range(x.shape[0])]
    for (a, b), cs in opp.items():
        ok = all(((x[c] - x[a]) * (x[c] - x[b])).sum() > 0 for c in cs)
        if ok:
            adj[a].append(b)
            adj[b].append(a)
    return adj


@pytest.mark.parametrize("gabriel_budget", [None, "0"], indirect=True)
def test_metrics_full_size_rmat18(G, gabriel_budget):
    """Random FP32 drawing of R-MAT 18: 64 sampled edges' crossings, the edge
    lengths, and every vertex's Jaccard index against a Delaunay-derived
    Gabriel graph."""
    g = inputs.rmat(18, 4, 0.57, 0.19, 0.19, seed=3)
    x = oracle.single(inputs.uniform_positions(g.n, seed=0, width=1200.0))
    out, ec, jac = _run(G, g, x, G.FP32)
    m = ec.size
    sel = np.random.default_rng(4).choice(m, 64, replace=False)
    assert np.array_equal(ec[sel], oracle.edge_crossings(g.n, g.row_ptr, g.col_idx, x, sel))
    assert out.crossings == int(ec.sum()) // 2
    assert out.crossings_per_edge == out.crossings / g.m
    once, _, _ = _run(G, g, x, G.FP32, what=G.METRIC_CROSSINGS, per_edge=False)
    assert once.crossings == out.crossings
    mu, sd = oracle.edge_lengths(g.n, g.row_ptr, g.col_idx, x)
    assert out.edge_length_mean == pytest.approx(mu, rel=1e-12)
    assert out.edge_length_std == pytest.approx(sd, rel=1e-10)
    adj = _delaunay_gabriel(x)
    expect = np.empty(g.n)
    for v in range(g.n):
        gn = set(adj[v])
        rn = set(g.col_idx[g.row_ptr[v]:g.row_ptr[v + 1]].tolist())
        uni = len(gn | rn)
        expect[v] = 1.0 if uni == 0 else len(gn & rn) / uni
    assert np.array_equal(jac, expect)
    assert out.gabriel_edges == sum(len(a) for a in adj) // 2
    print(f"rmat18 crossings={out.crossings} sim={out.similarity:.6f} gabriel={out.gabriel_edges}")


def _crossing_drawings():
    """Drawings at the edges of the crossing kernels: edge counts around one
    group (64) and around the count from which edges are sorted (4096), edges
    that cross whole groups, edges along one line, coincident points,
    coordinates whose squares leave float's range, and a flat drawing."""
    rng = np.random.default_rng(12)
    out = []
    for m in (1, 63, 64, 65, 4095, 4096, 4097, 4200):
        g = inputs.to_csr(2 * m, np.arange(m) * 2, np.arange(m) * 2 + 1)
        out.append((f"match{m}", g, rng.uniform(0.0, 100.0, (2 * m, 2))))
    # two bundles of 2100 nearly parallel edges, crossing each other at right angles
    m = 2100
    a = np.stack([rng.uniform(40, 60, m), rng.uniform(0, 1, m)], 1)
    b = np.stack([a[:, 0] + rng.uniform(-1, 1, m), rng.uniform(99, 100, m)], 1)
    x = np.concatenate([a, b, a[:, ::-1], b[:, ::-1]])
    e = np.arange(m)
    out.append(("bundles", inputs.to_csr(4 * m, np.concatenate([e, 2 * m + e]),
                                         np.concatenate([m + e, 3 * m + e])), x))
    g = inputs.erdos_renyi(900, 4500, seed=3)
    out.append(("line", g, np.stack([rng.integers(0, 50, g.n), 2.0 * rng.integers(0, 2, g.n)], 1).astype(float)))
    out.append(("coincident", g, rng.integers(0, 8, (g.n, 2)).astype(float)))
    y = rng.uniform(-1.0, 1.0, (g.n, 2))
    out += [("huge", g, y * 1e30), ("tiny", g, y * 1e-30), ("flat", g, y * np.array([1.0, 0.0])),
            ("far", g, y + 1e6)]
    return out


@pytest.mark.parametrize("i", range(15))
def test_crossings_at_kernel_edges(G, i):
    import torch
    name, g, x = _crossing_drawings()[i]
    print(f"crossings {name}", flush=True)
    x = oracle.single(x)
    rp, ci = G.to_device_csr(g)
    pos = torch.from_numpy(x.astype(np.float32)).cuda()
    per = torch.full((g.m,), -1, dtype=torch.int64, device="cuda")
    want = oracle.edge_crossings(g.n, g.row_ptr, g.col_idx, x, np.arange(g.m))
    total = G.drawing_metrics(rp, ci, G.FP32, pos, G.METRIC_CROSSINGS).crossings
    both = G.drawing_metrics(rp, ci, G.FP32, pos, G.METRIC_CROSSINGS, edge_crossings=per).crossings
    assert np.array_equal(per.cpu().numpy(), want)
    assert total == both == int(want.sum()) // 2


@pytest.mark.parametrize("n", [65536, 65537, 131072, 131073])
def test_similarity_by_eight_two_and_one_lanes(G, n, monkeypatch):
    """Where the number of lanes per point changes: the neighbours found by eight, two or one
    lane of each point, and by a wavefront of its own for every point
    (GILA_GABRIEL_BUDGET=0), are the same, at random, in clusters and on a lattice."""
    import torch
    g = inputs.erdos_renyi(n, 2 * n, seed=n)
    rp, ci = G.to_device_csr(g)
    rng = np.random.default_rng(n)
    at = {"random": rng.random((n, 2)) * 1000.0,
          "clusters": rng.integers(0, 200, (n, 2)) * 40.0 + rng.standard_normal((n, 2)),
          "lattice": np.stack([np.arange(n) % 300, np.arange(n) // 300], 1)}
    for name, x in at.items():
        print(f"similarity {name} n={n}", flush=True)
        pos = torch.from_numpy(x).float().cuda()
        found = []
        for budget in (None, "0"):
            if budget is None:
                monkeypatch.delenv("GILA_GABRIEL_BUDGET", raising=False)
            else:
                monkeypatch.setenv("GILA_GABRIEL_BUDGET", budget)
            jac = torch.zeros(n, dtype=torch.float64, device="cuda")
            m = G.drawing_metrics(rp, ci, G.FP32, pos, 4, None, jac)
            found.append((m.gabriel_edges, m.similarity, jac.cpu().numpy()))
        assert found[0][0] == found[1][0] > 0
        assert found[0][1] == found[1][1] and np.array_equal(found[0][2], found[1][2])
