"""Timed cases of the layout library: the calls a program makes, over the sizes it makes them at.

``listed()`` are the fixed cases and ``draw(rng)`` gives further ones of the same ranges.  Each
case names a call (``kind``), a graph family with its size, and the options of the layout:

  step      one iteration on a kept handle with its forces and moves (an interactive front end)
  run       a window of iterations on a kept handle (refining a drawing, resuming a layout)
  layout    lists built, a window of iterations run, handle released, in one call
  frame     lists built and one iteration: the first frame of a new graph
  pruned    the pipeline with degree-one vertices pruned and put back
  pack      connected components of a drawing, packed in a matrix
  batch     many small graphs: built and run in one launch
  batch_run the same on a kept batch handle
  metrics   crossings, edge lengths and Gabriel similarity of a drawing

The iterations run a late window of the cooling schedule from a seeded drawing, as refining or
resuming does.  A run from the schedule's start is chaotic (a rounding error grows a
hundredfold within two iterations), so two correct programs could not be compared on it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1606_02162_amd import gila, inputs

FRAME = 1200.0            # the paper's frame for the initial placement
D = gila.PAPER_IDEAL_LENGTH
WINDOW = 120              # first iteration of the window of the 0.93^h schedule
EXACT_PAIRS = 1 << 29     # cells of the reachability bitmap per chunk of the exact reference
PRECISIONS = {"fp64": gila.FP64, "fp32": gila.FP32, "fp32_kahan": gila.FP32_KAHAN}
MODELS = {"fr": (2, 1), "linlog": (0, 1), "p2q2": (2, 2)}


def listed():
    return [
        # the 32 x 32 mesh stepped one iteration at a time, forces returned: latency of one call
        {"name": "step_grid32_fp64", "kind": "step", "family": "grid", "n": 1024, "k": 2,
         "precision": "fp64", "model": "fr", "iterations": 1},
        # the same mesh refined: launches per iteration count
        {"name": "run_grid32_fp64", "kind": "run", "family": "grid", "n": 1024, "k": 2,
         "precision": "fp64", "model": "fr", "iterations": 20},
        # a small world of a serving size in one call: build and loop both count
        {"name": "layout_ws3k", "kind": "layout", "family": "ws", "n": 3001, "k": 3,
         "precision": "fp32_kahan", "model": "fr", "iterations": 50},
        # the Synth-Random shape under LinLog in double precision
        {"name": "run_er30k_linlog_fp64", "kind": "run", "family": "er", "n": 30011, "k": 3,
         "precision": "fp64", "model": "linlog", "iterations": 20},
        # the Synth-ScaleFree benchmark in one call
        {"name": "layout_ba100k_fp32", "kind": "layout", "family": "ba", "n": 100003, "k": 3,
         "precision": "fp32", "model": "fr", "iterations": 40},
        # the million-edge benchmark graph on a kept handle: the force kernel
        {"name": "run_rmat18", "kind": "run", "family": "rmat", "n": 262144, "k": 2,
         "precision": "fp32_kahan", "model": "fr", "iterations": 25},
        # a new million-edge graph until its first frame: the k-hop build
        {"name": "frame_rmat18", "kind": "frame", "family": "rmat", "n": 262144, "k": 2,
         "precision": "fp32_kahan", "model": "fr", "iterations": 1},
        # the paper's pipeline with pruning on a middle-sized power-law graph
        {"name": "pruned_rmat16", "kind": "pruned", "family": "rmat", "n": 65536, "k": 2,
         "precision": "fp32_kahan", "model": "fr", "iterations": 40},
        # a graph of many components arranged in a matrix
        {"name": "pack_rmat18", "kind": "pack", "family": "rmat", "n": 262144, "k": 0,
         "precision": "fp32_kahan", "model": "fr", "iterations": 0},
        # a quarter of the 4096-graph batch, from CSR to drawings
        {"name": "batch_1000_trees", "kind": "batch", "family": "trees", "n": 1000, "k": 3,
         "precision": "fp32", "model": "fr", "iterations": 50},
        # the largest graph of the serving workload, laid out in one call
        {"name": "layout_ws200k", "kind": "layout", "family": "ws", "n": 200000, "k": 2,
         "precision": "fp32_kahan", "model": "fr", "iterations": 40},
        # the quality measures of a half-million-edge drawing
        {"name": "metrics_rmat17", "kind": "metrics", "family": "rmat", "n": 131072, "k": 0,
         "precision": "fp32_kahan", "model": "fr", "iterations": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _graph_size(rng, family, most):
    if family == "rmat":
        return 1 << rng.randint(11, int(math.log2(most)))
    if family == "grid":
        return _log(rng, 12, math.sqrt(most)) ** 2
    return _log(rng, 200, most)


def draw(rng):
    kind = rng.choice(["step", "run", "run", "run", "layout", "layout", "layout", "frame", "pruned",
                       "pack", "batch", "batch_run", "metrics", "metrics"])
    c = {"kind": kind, "precision": rng.choice(["fp64", "fp32", "fp32_kahan", "fp32_kahan"]),
         "model": "fr", "iterations": rng.randint(10, 40)}
    if kind in ("batch", "batch_run"):
        return {**c, "family": "trees", "n": _log(rng, 8, 1500), "k": rng.choice([2, 3])}
    if kind in ("pack", "metrics"):
        family = rng.choice(["grid", "ws", "ba", "er", "rmat"])
        most = {"grid": 200000, "ws": 150000, "ba": 90000, "er": 110000, "rmat": 65536}[family]
        return {**c, "family": family, "n": _graph_size(rng, family, most), "k": 0,
                "iterations": 0}
    family = rng.choice(["grid", "ws", "ba", "er", "rmat", "tree"])
    most = {"grid": 250000, "ws": 200000, "ba": 60000, "er": 150000, "rmat": 131072,
            "tree": 100000}[family]
    k = 2 if family == "rmat" else rng.choice([2, 3])
    if kind in ("step", "run", "layout"):
        c["model"] = rng.choice(["fr", "fr", "linlog", "p2q2"])
    if kind in ("step", "frame"):
        c["iterations"] = 1
    if kind == "pruned":
        family, k, most = rng.choice([("rmat", 2, 65536), ("tree", 3, 60000), ("er", 3, 60000)])
    return {**c, "family": family, "n": _graph_size(rng, family, most), "k": k}


# ------------------------------------------------------------------ inputs
def _sizes(case):
    """Vertex counts of the graphs of a batch (the benchmark's size seed)."""
    return inputs.log_uniform_sizes(case["n"], 50, 5000, 4)


def _trees(sizes, seed):
    """Block-diagonal CSR of random recursive trees with n // 2 extra random edges each (the
    shape of ``inputs.random_tree_plus_edges``, thousands of graphs at once)."""
    rng = np.random.default_rng(seed)
    base = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    local = np.arange(int(sizes.sum())) - np.repeat(base, sizes)
    own = np.repeat(base, sizes)
    parent = own + np.floor(rng.random(local.size) * np.maximum(local, 1)).astype(np.int64)
    child = own + local
    keep = local > 0
    extra = sizes // 2
    eb, en = np.repeat(base, extra), np.repeat(sizes, extra)
    a = eb + np.floor(rng.random(eb.size) * en).astype(np.int64)
    b = eb + np.floor(rng.random(eb.size) * en).astype(np.int64)
    return inputs.to_csr(int(sizes.sum()), np.concatenate([child[keep], a]),
                         np.concatenate([parent[keep], b])), base


def _graph(case, seed):
    family, n = case["family"], case["n"]
    if family == "grid":
        # a mesh has no randomness of its own: the seed gives its drawing
        return inputs.grid_graph(int(round(math.sqrt(n))), int(round(math.sqrt(n))))
    if family == "ws":
        return inputs.watts_strogatz(n, 6, 0.1, seed)
    if family == "ba":
        return inputs.barabasi_albert(n, 3, seed)
    if family == "er":
        return inputs.erdos_renyi(n, (5 * n) // 2, seed)
    if family == "rmat":
        return inputs.rmat(int(round(math.log2(n))), 4, 0.57, 0.19, 0.19, seed)
    if family == "tree":
        return _trees(np.array([n]), seed)[0]
    raise ValueError(family)


def _smooth(g, x, rounds=12):
    """A drawing with short edges, as a finished layout has: positions averaged over the
    neighbours, then spread evenly over the frame coordinate by coordinate."""
    deg = np.maximum(g.degrees(), 1)[:, None]
    some = g.degrees() > 0
    starts = g.row_ptr[:-1][some]
    for _ in range(rounds):
        s = np.zeros_like(x)
        s[some] = np.add.reduceat(x[g.col_idx], starts, axis=0)
        x = np.where(some[:, None], 0.5 * x + 0.5 * s / deg, x)
    out = np.empty_like(x)
    for c in range(2):
        out[np.argsort(x[:, c], kind="stable"), c] = (np.arange(g.n) + 0.5) * (FRAME / g.n)
    return out


def _positions(case, seed, g):
    x = inputs.uniform_positions(g.n, seed, FRAME)
    if case["kind"] in ("metrics", "pack"):
        x = _smooth(g, x)
    return x if case["precision"] == "fp64" else x.astype(np.float32)


def _window(case, n):
    """The caps of the case's window of the paper's schedule for n vertices."""
    it = case["iterations"]
    return gila.paper_schedule(max(n, 1), 1.0, D, WINDOW + it)


def _params(case, n, temps=None):
    p, q = MODELS[case["model"]]
    return gila.LayoutParams(temperature=_window(case, n) if temps is None else temps,
                             precision=PRECISIONS[case["precision"]],
                             stop_fraction=0.15 if case["kind"] == "layout" else 0.0,
                             force_model=gila.MODEL_FR if case["model"] == "fr" else gila.MODEL_PQ,
                             force_p=p, force_q=q)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("batch", "batch_run"):
        sizes = _sizes(case)
        g, base = _trees(sizes, seed)
        # each graph's rows counted from 0 and in its own ids, one after another
        rp = np.concatenate([g.row_ptr[b:b + n + 1] - g.row_ptr[b] for b, n in zip(base, sizes)])
        nnz = g.row_ptr[base + sizes] - g.row_ptr[base]
        s["rp"], s["ci"] = _dev(rp), _dev(g.col_idx - np.repeat(base, nnz).astype(np.int32))
        s["n"], s["nnz"], s["base"] = sizes, nnz, base
        s["pos0"] = _dev(_positions(case, seed, g))
        s["pos"] = torch.empty_like(s["pos0"])
        s["params"] = gila.BatchParams([_window(case, int(n))[WINDOW:] for n in sizes],
                                       precision=PRECISIONS[case["precision"]])
        if kind == "batch_run":
            s["batch"] = gila.Batch.concatenated(s["rp"], s["ci"], sizes, nnz, case["k"])
        return s
    g = _graph(case, seed)
    s["rp"], s["ci"] = gila.to_device_csr(g)
    s["pos0"] = _dev(_positions(case, seed, g))
    s["pos"] = torch.empty_like(s["pos0"])
    s["params"] = _params(case, g.n)
    if kind in ("layout", "pruned"):  # these run all of a schedule: the window alone
        s["params"] = _params(case, g.n, _window(case, g.n)[WINDOW:])
    if kind in ("step", "run"):
        s["kh"] = gila.build_khop(s["rp"], s["ci"], case["k"])
    if kind == "step":
        s["force"] = torch.empty((g.n, 2), dtype=torch.float64, device="cuda")
        s["disp"] = torch.empty_like(s["force"])
    if kind == "metrics":
        # room for four edges per vertex, whatever the seed's count: the call writes the first m
        s["edge"] = torch.zeros(4 * g.n, dtype=torch.int64, device="cuda") if case["n"] < 50000 else None
        s["jaccard"] = torch.empty(g.n, dtype=torch.float64, device="cuda")
    return s


# ------------------------------------------------------------------ one pass
def _stats(st):
    return {"iterations": st.iterations_run, "moved": st.moved, "coincident": st.coincident,
            "max_disp": st.max_disp, "energy": st.energy}


def _all_stats(sts, single):
    """Statistics of many graphs, the measured values in the precision of their layout."""
    f = np.float32 if single else np.float64
    return {"iterations": np.array([st.iterations_run for st in sts], dtype=np.int64),
            "moved": np.array([st.moved for st in sts], dtype=np.int64),
            "coincident": np.array([st.coincident for st in sts], dtype=np.int64),
            "max_disp": np.array([st.max_disp for st in sts], dtype=f),
            "energy": np.array([st.energy for st in sts], dtype=f)}


def run(s):
    case = s["case"]
    kind, single = case["kind"], case["precision"] != "fp64"
    pos = s["pos"]
    pos.copy_(s["pos0"])
    if kind in ("batch", "batch_run"):
        b = s.get("batch") or gila.Batch.concatenated(s["rp"], s["ci"], s["n"], s["nnz"], case["k"])
        st = b.run(s["params"], (pos, s["base"]))
        if kind == "batch":
            b.free()
        return {"pos": pos, **_all_stats(st, single)}
    if kind == "step":
        out = {}
        st = gila.step(s["kh"], s["params"], WINDOW, pos, s["force"], s["disp"])
        if not single:  # in single precision these are single-precision sums, widened
            out = {"force": s["force"], "disp": s["disp"]}
        return {"pos": pos, **out, **_stats(st)}
    if kind == "run":
        st = gila.run(s["kh"], s["params"], pos, start_h=WINDOW)
        return {"pos": pos, **_stats(st)}
    if kind == "layout":
        return {"pos": pos, **_stats(gila.layout(s["rp"], s["ci"], case["k"], s["params"], pos))}
    if kind == "frame":
        kh = gila.build_khop(s["rp"], s["ci"], case["k"])
        pairs = kh.info()["total_pairs"]
        st = gila.step(kh, s["params"], WINDOW, pos)
        kh.free()
        return {"pos": pos, "pairs": pairs, **_stats(st)}
    if kind == "pruned":
        return {"pos": pos, **_stats(gila.layout_pruned(s["rp"], s["ci"], case["k"], s["params"], pos))}
    precision = PRECISIONS[case["precision"]]
    if kind == "pack":
        label, count = gila.components(s["rp"], s["ci"])
        gila.pack_components(label, D, precision, pos)
        return {"pos": pos, "label": label, "count": count}
    m = gila.drawing_metrics(s["rp"], s["ci"], precision, pos, edge_crossings=s["edge"],
                             jaccard=s["jaccard"])
    return {**m.as_dict(), "edge": s["edge"], "jaccard": s["jaccard"]}


# ------------------------------------------------------------------ 64-bit reference
class _Lists:
    """N_v(k) of every vertex (or of the given ones) by breadth-first search in torch."""

    def __init__(self, row_ptr, col_idx, k, base=None, width=None, rows=None):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.rp = torch.from_numpy(np.ascontiguousarray(row_ptr)).to(dev)
        self.ci = torch.from_numpy(np.ascontiguousarray(col_idx)).to(dev).long()
        n = self.rp.numel() - 1
        self.n = n
        # column of vertex u in the bitmap row of v: u - base[v] (base: its graph's first id)
        self.base = torch.zeros(n, dtype=torch.long, device=dev) if base is None else \
            torch.from_numpy(base).to(dev)
        width = n if width is None else width
        some = torch.nonzero(self.rp[1:] > self.rp[:-1]).flatten() if rows is None else \
            torch.from_numpy(rows).to(dev)
        self.chunks = []
        step = max(1, EXACT_PAIRS // max(width, 1))
        for i in range(0, some.numel(), step):
            v = some[i:i + step]
            at = torch.arange(v.numel(), device=dev)
            mark = torch.zeros((v.numel(), width), dtype=torch.bool, device=dev)
            mark[at, v - self.base[v]] = True
            r, u = at, v
            for level in range(k):
                rr, w = self._expand(r, u)
                new = torch.zeros_like(mark) if level + 1 < k else mark
                new[rr, w - self.base[v][rr]] = True
                if level + 1 < k:
                    new &= ~mark
                    mark |= new
                    r, c = torch.nonzero(new, as_tuple=True)
                    u = c + self.base[v][r]
                del rr, w, new
            mark[at, v - self.base[v]] = False
            r, c = torch.nonzero(mark, as_tuple=True)
            self.chunks.append((v, r.int(), (c + self.base[v][r]).int(),
                                torch.searchsorted(r, torch.arange(1, v.numel() + 1, device=dev))))
            del mark
        self.pairs = sum(r.numel() for _, r, _, _ in self.chunks)
        # the row of each adjacency entry
        self.src = torch.repeat_interleave(torch.arange(n, device=dev), self.rp[1:] - self.rp[:-1])

    def _expand(self, r, u):
        deg = self.rp[u + 1] - self.rp[u]
        end = torch.cumsum(deg, 0)
        at = torch.arange(int(end[-1]) if end.numel() else 0, device=u.device)
        at += torch.repeat_interleave(self.rp[u] - (end - deg), deg)
        return torch.repeat_interleave(r, deg), self.ci[at]


def _row_sums(end, terms):
    """Sums over the rows of the terms [m, 2], row i's ending before end[i]; [rows, 2]."""
    out = []
    for col in terms.unbind(1):
        run = torch.cumsum(col.contiguous(), 0)
        total = torch.cat([run.new_zeros(1), run])[end]
        out.append(total - torch.cat([total.new_zeros(1), total[:-1]]))
    return torch.stack(out, 1)


def _forces(lists, x, model, mass=None):
    p, q = MODELS[model]
    force = torch.zeros_like(x)
    coincident = 0
    for v, r, u, end in lists.chunks:
        r, u = r.long(), u.long()
        dx = x[v][r] - x[u]
        d2 = (dx * dx).sum(1)
        far = d2 > 0
        coincident += int((~far).sum())
        f = torch.where(far, D * D * torch.where(far, d2, torch.ones_like(d2)) ** (-(q + 1) / 2),
                        torch.zeros_like(d2))
        if mass is not None:
            f = f * mass[u]
        force[v] += _row_sums(end, dx * f[:, None])
    dx = x[lists.ci] - x[lists.src]
    d2 = (dx * dx).sum(1)
    far = d2 > 0
    f = torch.where(far, torch.where(far, d2, torch.ones_like(d2)) ** ((p - 1) / 2) / D,
                    torch.zeros_like(d2))
    force += _row_sums(lists.rp[1:], dx * f[:, None])
    return force, coincident


def _iterate(lists, x, model, temps, mass=None, stop=0.0, part=None, parts=1):
    """Iterations with the caps temps [h][parts] of each graph; part: the graph of each vertex.
    Returns the drawing and, per graph, the last iteration's statistics."""
    dev = x.device
    part = torch.zeros(lists.n, dtype=torch.long, device=dev) if part is None else part
    active = lists.rp[1:] > lists.rp[:-1]
    n_active = torch.bincount(part[active], minlength=parts)
    going = torch.ones(parts, dtype=torch.bool, device=dev)
    zero = torch.zeros(parts, dtype=torch.float64, device=dev)
    st = {"iterations": zero.long(), "moved": zero.long(), "coincident": zero.long(),
          "max_disp": zero.clone(), "energy": zero.clone()}
    force = disp = torch.zeros_like(x)
    for t in temps:
        force, coincident = _forces(lists, x, model, mass)
        size = torch.sqrt((force * force).sum(1))
        cap = torch.as_tensor(t, dtype=torch.float64, device=dev).reshape(-1)[part]
        disp = force * torch.where(size > 0, torch.minimum(size, cap) / size, torch.zeros_like(size))[:, None]
        disp = torch.where(going[part][:, None], disp, torch.zeros_like(disp))
        x = x + disp
        move = torch.sqrt((disp * disp).sum(1))
        now = {"moved": torch.bincount(part, weights=(move > 0.01).double(), minlength=parts).long(),
               "coincident": torch.full_like(zero, coincident).long(),
               "max_disp": zero.clone().scatter_reduce(0, part, move, "amax"),
               "energy": torch.bincount(part, weights=size * size, minlength=parts)}
        st["iterations"] += going.long()
        for key, val in now.items():
            st[key] = torch.where(going, val, st[key])
        if stop > 0:
            going = going & ~(now["moved"] < stop * n_active)
    return x, force, disp, {key: val.cpu().numpy() for key, val in st.items()}


def _exact_pruned(case, g, x, temps):
    """Pruning, weighted iterations and reinsertion with plain numpy around _iterate."""
    deg, src = g.degrees(), np.repeat(np.arange(g.n), g.degrees())
    only = np.where(deg == 1, g.col_idx[np.minimum(g.row_ptr[:-1], max(g.nnz - 1, 0))], -1)
    gone = (deg == 1) & ~((deg[only] == 1) & (only > np.arange(g.n)))
    leaves = np.bincount(only[gone], minlength=g.n)
    keep = np.nonzero(~gone)[0]
    new = np.full(g.n, -1)
    new[keep] = np.arange(keep.size)
    e = ~gone[src] & ~gone[g.col_idx]
    u, v = new[src[e]], new[g.col_idx[e]]
    rp = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=keep.size))])
    lists = _Lists(rp, v, case["k"])
    mass = torch.from_numpy(1.0 + leaves[keep]).to(lists.rp.device)
    y, _, _, st = _iterate(lists, torch.from_numpy(x[keep]).to(lists.rp.device), "fr", temps, mass)
    y = y.cpu().numpy()
    out = np.zeros_like(x)
    out[keep] = y
    order = np.argsort(only[gone], kind="stable")
    hung, anchor = np.nonzero(gone)[0][order], only[gone][order]
    first = np.concatenate([[0], np.cumsum(leaves)])
    for a in np.nonzero(leaves)[0]:
        mine, count = hung[first[a]:first[a + 1]], int(leaves[a])
        near = y[v[rp[new[a]]:rp[new[a] + 1]]] - y[new[a]]
        phi, rho = 0.0, 0.2 * D
        if near.size:
            rho = 0.2 * float(np.sqrt((near * near).sum(1)).min())
            period = 2 * math.pi / count
            res = np.sort(np.mod(np.arctan2(near[:, 1], near[:, 0]), period))
            gap = np.diff(np.concatenate([res, [res[0] + period]]))
            i = int(np.argmax(gap))
            phi = math.fmod(res[i] + 0.5 * gap[i], period)
        ang = phi + 2 * math.pi * np.arange(count) / count
        out[mine] = y[new[a]] + rho * np.stack([np.cos(ang), np.sin(ang)], 1)
    return {"pos": out, **{key: None for key in ("iterations", "moved", "coincident")},
            "max_disp": float(st["max_disp"][0]), "energy": float(st["energy"][0])}


def _exact_pack(g, x):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    label = torch.arange(g.n, device=dev)
    src = torch.from_numpy(np.repeat(np.arange(g.n), g.degrees())).to(dev)
    dst = torch.from_numpy(g.col_idx).to(dev).long()
    while True:
        low = label.scatter_reduce(0, src, label[dst], "amin")
        low = low[low]
        if torch.equal(low, label):
            break
        label = low
    label = label.cpu().numpy()
    ids, comp, size = np.unique(label, return_inverse=True, return_counts=True)
    order = np.lexsort((ids, -size))
    rank = np.empty_like(order)
    rank[order] = np.arange(order.size)
    rank = rank[comp]
    lo, hi = np.full((ids.size, 2), np.inf), np.full((ids.size, 2), -np.inf)
    np.minimum.at(lo, rank, x)
    np.maximum.at(hi, rank, x)
    cols = int(math.ceil(math.sqrt(ids.size)))
    cell = np.arange(ids.size)
    width, height = np.zeros(cols), np.zeros(-(-ids.size // cols))
    np.maximum.at(width, cell % cols, (hi - lo)[:, 0])
    np.maximum.at(height, cell // cols, (hi - lo)[:, 1])
    left = np.concatenate([[0], np.cumsum(width + D)[:-1]])
    low = np.concatenate([[0], np.cumsum(height + D)[:-1]])
    corner = np.stack([left[cell % cols], low[cell // cols]], 1)
    return {"pos": x - lo[rank] + corner[rank], "label": None, "count": None}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "batch_run"):
        sizes = _sizes(case)
        g, base = _trees(sizes, seed)
        lists = _Lists(g.row_ptr, g.col_idx, case["k"], np.repeat(base, sizes), int(sizes.max()))
        x = _round(case, inputs.uniform_positions(g.n, seed, FRAME)).to(lists.rp.device)
        part = torch.from_numpy(np.repeat(np.arange(sizes.size), sizes)).to(x.device)
        temps = np.stack([_caps(case, int(n)) for n in sizes], 1)
        y, _, _, st = _iterate(lists, x, "fr", temps, part=part, parts=sizes.size)
        return {"pos": y, "iterations": None, "moved": None, "coincident": None,
                "max_disp": st["max_disp"], "energy": st["energy"]}
    g = _graph(case, seed)
    x = _positions(case, seed, g).astype(np.float64)
    if kind == "metrics":
        x = x.astype(np.float32).astype(np.float64)  # the measures are those of the single-precision drawing
        e = g.edges()
        length = np.sqrt(((x[e[:, 0]] - x[e[:, 1]]) ** 2).sum(1))
        return {**{key: None for key in ("edges", "crossings", "similarity", "gabriel_edges", "edge",
                                         "jaccard")},
                "edge_length_mean": float(length.mean()) if e.size else 0.0,
                "edge_length_std": float(length.std()) if e.size else 0.0}
    if kind == "pack":
        return _exact_pack(g, x)
    temps = _caps(case, g.n)
    if kind == "pruned":
        return _exact_pruned(case, g, x, temps)
    lists = _Lists(g.row_ptr, g.col_idx, case["k"])
    y, force, disp, st = _iterate(lists, torch.from_numpy(x).to(lists.rp.device), case["model"], temps,
                                  stop=0.15 if kind == "layout" else 0.0)
    out = {"pos": y, "iterations": None, "moved": None, "coincident": None, "pairs": None,
           "max_disp": float(st["max_disp"][0]), "energy": float(st["energy"][0])}
    if kind == "step" and case["precision"] == "fp64":
        out |= {"force": force, "disp": disp}
    return out


def _round(case, x):
    return torch.from_numpy(x if case["precision"] == "fp64" else x.astype(np.float32).astype(np.float64))


def _caps(case, n):
    return _window(case, n)[WINDOW:]


# ------------------------------------------------------------------ what a pass cannot do without
def _pairs(g, k, base=None, width=None):
    """sum |N_v(k)|, estimated from at most 512 vertices."""
    some = np.nonzero(g.degrees())[0]
    if not some.size:
        return 0.0
    rows = some[:: max(1, some.size // 512)]
    lists = _Lists(g.row_ptr, g.col_idx, k, base, width, rows)
    return lists.pairs * (some.size / rows.size)


def work(case):
    """The graph read once, positions read and written once, and per iteration one id of four bytes
    and about ten operations for each pair and each adjacency entry; for the measures the sign
    tests of the pairs of edges that a sweep cannot rule out are not counted, only the edges."""
    kind, it = case["kind"], max(case["iterations"], 1)
    if kind in ("batch", "batch_run"):
        sizes = _sizes(case)
        g, base = _trees(sizes, 1)
        n, nnz = g.n, g.nnz
        pairs = _pairs(g, case["k"], np.repeat(base, sizes), int(sizes.max()))
    else:
        g = _graph(case, 1)
        n, nnz = g.n, g.nnz
        pairs = _pairs(g, case["k"]) if case["k"] else 0.0
    pos = (32 if case["precision"] == "fp64" else 16) * n
    graph = 8 * n + 4 * nnz
    if kind in ("pack", "metrics"):
        return {"bytes": float(graph + pos + 8 * n), "flops": float(40 * nnz + 10 * n)}
    return {"bytes": float(graph + pos + it * (4 * pairs + 4 * nnz + pos)),
            "flops": float(it * 10 * (pairs + nnz))}
