"""The force kernel's division of work: rows of every length side by side (each is
walked by the lanes that its own length asks for), in one workgroup, in the default
number of them and in as many as the smallest share allows, against the FP64 oracle.

Gates as for one step: forces and positions within 1e-12 in FP64 and 1e-5 in FP32.
"""
import numpy as np
import pytest

import oracle
from gpu_common import oracle_rows, pos_err, rel_l2, require_gpu
from paper_1606_02162_amd import inputs

pytestmark = pytest.mark.gpu


def _cliques_and_path(path):
    """Cliques of 2 to 1025 vertices (rows of 1, 3, 4, 15, 16, ... 1024 ids) and a path."""
    edges, base = [], 0
    for size in (2, 4, 5, 16, 17, 33, 64, 65, 129, 257, 513, 1025):
        i, j = np.triu_indices(size, 1)
        edges.append(np.stack([i + base, j + base], 1))
        base += size
    if path:
        i = np.arange(base, base + path - 1)
        edges.append(np.stack([i, i + 1], 1))
    u, v = np.concatenate(edges).T
    return inputs.to_csr(base + path, u, v, f"cliques+{path}")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_kahan"])
@pytest.mark.parametrize("path", [0, 9001])
@pytest.mark.parametrize("workgroups", ["1", "0", "4096"])
def test_rows_of_every_length(precision, path, workgroups, monkeypatch):
    require_gpu()
    import torch
    from paper_1606_02162_amd import gila
    monkeypatch.setenv("GILA_SEG_WG", workgroups)
    g = _cliques_and_path(path)
    prec = gila.PRECISIONS[precision]
    pos0 = inputs.uniform_positions(g.n, seed=5, width=1500.0).astype(np.float32).astype(np.float64)
    rp, ci = gila.to_device_csr(g)
    kh = gila.build_khop(rp, ci, 1)
    params = gila.LayoutParams(temperature=np.array([20.0]), ideal_length=30.0, precision=prec)
    pos = torch.from_numpy(pos0).to(dtype=gila.position_dtype(prec), device="cuda")
    F = torch.zeros((g.n, 2), dtype=torch.float64, device="cuda")
    D = torch.zeros((g.n, 2), dtype=torch.float64, device="cuda")
    gila.step(kh, params, 0, pos, F, D)
    kh.free()
    optr, oidx = oracle_rows(g, 1)
    x, Fo, _, _ = oracle.step(g.n, g.row_ptr, g.col_idx, optr, oidx, 30.0, 20.0, pos0)
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert rel_l2(F.cpu().numpy(), Fo) <= tol
    assert pos_err(pos.double().cpu().numpy(), x) <= tol
