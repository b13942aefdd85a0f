"""Edges of the network kernels' row tiles against the FP64 network oracle.

The forward pass works on pairs of 32-row tiles, one pair per wave, on a grid that wraps after
131072 rows.  Each row's result depends on that row alone, and one tile's sums have the same order
wherever the row lies.  Rows are compared as in test_gpu_mlp.py: the 99th percentile of the
row error within 1e-4 of the largest output (FP32 against FP64 sums), the worst within 1e-2 (values
that round to the other bfloat16 neighbour).
"""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


def _net(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for _, s in M.SHAPES:
        k = int(np.prod(s))
        parts.append(rng.uniform(-1, 1, k) * (np.sqrt(6.0 / s[-1]) if len(s) == 2 else 0.2))
    return np.concatenate(parts).astype(np.float32)


@pytest.mark.parametrize("n", [32, 33, 64, 65, 131105])
def test_forward_rows_at_tile_edges(n):
    import torch
    from paper_2604_17513_amd import flash as F
    th = _net(5)
    X = np.random.default_rng(n).standard_normal((n, 16)).astype(np.float32)
    m = F.Mlp(max_rows=64, seed=0)
    m.set_params(th)
    yd = torch.full((n + 1, 3), 7.0, dtype=torch.float32, device="cuda")
    m.forward(torch.from_numpy(X).cuda(), n, yd)
    Y = yd.cpu().numpy().astype(np.float64)
    R, _ = M.forward(th.astype(np.float64), X.astype(np.float64), rounded=True)
    err = np.abs(Y[:n] - R).max(axis=1) / np.abs(R).max()
    print(f"n={n}: p99 {np.percentile(err, 99):.2e} max {err.max():.2e}", flush=True)
    assert np.percentile(err, 99) <= 1e-4 and err.max() <= 1e-2
    assert np.all(Y[n] == 7.0)            # nothing past the last row
    # one bad row stays its own affair
    X[n // 2, 3] = np.nan
    m.forward(torch.from_numpy(X).cuda(), n, yd)
    Z = yd.cpu().numpy()[:n].astype(np.float64)
    others = np.arange(n) != n // 2
    assert np.array_equal(Z[others], Y[:n][others])


@pytest.mark.parametrize("n", [1, 127, 128, 129, 32897])
def test_gradient_at_row_blocks(n):
    """Blocks of 128 rows per workgroup, a partial last one, and more blocks than the grid's 256
    workgroups (32897 rows: two workgroups take a second block).  Tolerances of test_gpu_mlp.py's
    gradient test: norm-wise 1e-2 overall, 2e-2 per parameter block."""
    import torch
    from paper_2604_17513_amd import flash as F
    th = _net(6)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 16)).astype(np.float32)
    T = rng.standard_normal((n, 3)).astype(np.float32)
    m = F.Mlp(max_rows=n, seed=0)
    m.set_params(th)
    g, loss = m.grad(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), n)
    L, gr = M.loss_and_grad(th.astype(np.float64), X.astype(np.float64), T.astype(np.float64), rounded=True)
    print(f"n={n}: loss {loss:.6e} / {L:.6e}, grad {np.linalg.norm(g - gr) / np.linalg.norm(gr):.2e}", flush=True)
    assert abs(loss - L) <= 2e-3 * L
    assert np.linalg.norm(g - gr) <= 1e-2 * np.linalg.norm(gr)
    off = 0
    for name, shp in M.SHAPES:
        k = int(np.prod(shp))
        blk = slice(off, off + k)
        off += k
        assert np.linalg.norm(g[blk] - gr[blk]) <= 2e-2 * np.linalg.norm(gr[blk]) + 1e-6 * np.linalg.norm(gr), name
