"""The halting rule where an iteration's statistics are reduced beside the next
one's forces: runs that stop at their first, a middle and their last
iteration, on one-segment and many-segment graphs, in one captured range, in
chunks and in split runs, against single steps whose statistics decide on the
host.  The same kernels in the same order: the same bits."""
import os

import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu
PATHS = {"one_segment": {}, "segments": {"GILA_SEG_BYTES": "2048"},
         "dense": {"GILA_DENSE_MIN": "1"}, "direct": {"GILA_PATH": "direct"}}


@pytest.fixture(params=list(PATHS))
def path(request, monkeypatch):
    for k, v in PATHS[request.param].items():
        monkeypatch.setenv(k, v)
    return request.param


@pytest.fixture(scope="module")
def G():
    require_gpu()
    from paper_1606_02162_amd import gila
    return gila


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_kahan"])
@pytest.mark.parametrize("H,stop", [(1, 0), (6, 0), (6, 1), (7, 3), (7, 6), (7, None), (130, 101),
                                    (130, 99), (130, None)])
def test_stops_where_single_steps_do(G, path, precision, H, stop):
    import torch
    print(f"halting {path} {precision} H={H} stop={stop}", flush=True)
    g = inputs.erdos_renyi(300, 800, seed=1)
    rp, ci = G.to_device_csr(g)
    prec = G.PRECISIONS[precision]
    # every vertex moves by the cap until iteration `stop`, whose cap is below the threshold
    temps = np.full(H, 0.5)
    if stop is not None:
        temps[stop] = 0.001
    params = G.LayoutParams(temperature=temps, precision=prec, stop_fraction=0.5)
    x = torch.from_numpy(inputs.uniform_positions(g.n, 3)).to(dtype=G.position_dtype(prec), device="cuda")
    kh = G.build_khop(rp, ci, 2)
    kh.enable_history(H)
    ref, rows, ran = x.clone(), [], 0
    for h in range(H):
        st = G.step(kh, params, h, ref)
        rows.append((st.energy, st.max_disp, float(st.moved), float(st.coincident)))
        ran += 1
        if stop is not None and h == stop:
            break
    kh.enable_history(H)
    pos = x.clone()
    st = G.run(kh, params, pos)
    assert st.iterations_run == ran and st.stopped == (1 if stop is not None else 0)
    assert torch.equal(pos, ref)
    assert (st.energy, st.max_disp, float(st.moved), float(st.coincident)) == rows[-1]
    hist = kh.history(0, H)
    assert np.array_equal(hist[:ran], np.array(rows)) and np.isnan(hist[ran:]).all()
    # split at an odd place: the same bits
    pos = x.clone()
    cut = min(3, H)
    a = G.run(kh, params, pos, 0, cut)
    if not a.stopped and cut < H:
        G.run(kh, params, pos, cut, H)
    assert torch.equal(pos, ref)


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("H,stop", [(7, 3), (130, 70)])
def test_stops_with_more_workgroups_than_the_device_holds(G, precision, H, stop, monkeypatch):
    """4096 workgroups a launch, of which at most 1024 are resident: some of the launch after
    the last iteration begin while, or after, its first workgroup sets the flag that they
    read.  As above: the bits of single steps (the longer run in replayed chunks)."""
    import torch
    print(f"halting 4096 workgroups {precision} H={H} stop={stop}", flush=True)
    monkeypatch.setenv("GILA_SEG_WG", "4096")
    g = inputs.barabasi_albert(20000, 3, seed=4)
    rp, ci = G.to_device_csr(g)
    prec = G.PRECISIONS[precision]
    temps = np.full(H, 0.5)
    temps[stop] = 0.001
    params = G.LayoutParams(temperature=temps, precision=prec, stop_fraction=0.5)
    x = torch.from_numpy(inputs.uniform_positions(g.n, 3)).to(dtype=G.position_dtype(prec), device="cuda")
    kh = G.build_khop(rp, ci, 3)
    ref = x.clone()
    for h in range(stop + 1):
        last = G.step(kh, params, h, ref)
    pos = x.clone()
    st = G.run(kh, params, pos)
    assert st.iterations_run == stop + 1 and st.stopped == 1
    assert (st.energy, st.max_disp, st.moved, st.coincident) == \
        (last.energy, last.max_disp, last.moved, last.coincident)
    assert torch.equal(pos, ref)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_coincident_pairs_are_counted_for_their_own_iteration(G, path, precision):
    """Twins (four leaves of each vertex of a path, in one place) stay coincident: every
    iteration counts the same pairs while it reduces the one before.  In one range, in
    replayed chunks and in single steps."""
    import torch
    print(f"coincident {path} {precision}", flush=True)
    hubs, H = 2000, 110
    i = np.arange(hubs)
    leaf = hubs + 4 * i[:, None] + np.arange(4)[None, :]
    u = np.concatenate([i[:-1], np.repeat(i, 4)])
    v = np.concatenate([i[1:], leaf.ravel()])
    g = inputs.to_csr(5 * hubs, u, v, "twins")
    x = inputs.uniform_positions(g.n, 3)
    x[leaf] = x[leaf[:, :1]]
    rp, ci = G.to_device_csr(g)
    prec = G.PRECISIONS[precision]
    params = G.LayoutParams(temperature=np.full(H, 0.5), precision=prec)
    x = torch.from_numpy(x).to(dtype=G.position_dtype(prec), device="cuda")
    kh = G.build_khop(rp, ci, 2)
    pairs = 12 * hubs  # ordered pairs of four twins
    for end in (3, 20, H):
        kh.enable_history(H)
        pos = x.clone()
        st = G.run(kh, params, pos, 0, end)
        assert st.iterations_run == end and st.coincident == pairs
        assert (kh.history(0, end)[:, 3] == pairs).all()
    ref = x.clone()
    for h in range(5):
        assert G.step(kh, params, h, ref).coincident == pairs
