"""The reparameterisation solve on graphs whose rows differ from a mesh's: more
neighbours than the solve's table holds, none at all, single vertices, an odd
last iteration, a large lambda."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


def _graph(nv, edges):
    A = np.zeros((nv, nv))
    for i, j in edges:
        A[i, j] = A[j, i] = 1.0
    off = np.concatenate([[0], np.cumsum(A.sum(1))]).astype(np.int32)
    adj = np.concatenate([np.flatnonzero(r) for r in A] + [np.zeros(0, int)]).astype(np.int32)
    return A, off, adj


def _case(kind):
    if kind == "single":
        return 1, []
    if kind == "star":      # one vertex of degree 40, forty of degree 1
        return 41, [(0, i) for i in range(1, 41)]
    if kind == "degree9":   # rows just past the table's 8
        return 20, [(i, j) for i in range(10) for j in range(i)] + [(i, i + 1) for i in range(9, 18)]
    return 515, [(i, i + 1) for i in range(0, 512)]   # a path, and two loose vertices


@pytest.mark.parametrize("kind", ["single", "star", "degree9", "path"])
@pytest.mark.parametrize("lam", [3.0, 1e4])
def test_rows_against_the_dense_solve(kind, lam):
    dev = device()
    nv, edges = _case(kind)
    A, off, adj = _graph(nv, edges)
    M = np.eye(nv) + lam * (np.diag(A.sum(1)) - A)
    b = np.random.default_rng(nv).normal(size=(nv, 3))
    ref = np.linalg.solve(M, b)
    # an empty list still needs an array to point at
    adj = adj if len(adj) else np.zeros(1, np.int32)
    s = B.Smooth(torch.from_numpy(off).to(dev), torch.from_numpy(adj).to(dev), lam)
    x = torch.zeros(nv, 3, dtype=torch.float64, device=dev)
    s.solve(torch.from_numpy(b).to(dev), x, max_iters=20000)
    got = x.cpu().numpy()
    # |error| <= |residual| (the smallest eigenvalue is 1): 1e-10 of |b| a column
    # and the residual's own rounding, 20 u (1 + lam m)
    m = max([1.0] + [A[i].sum() + (A[i] @ A.sum(1)) / A[i].sum() for i in range(nv) if A[i].any()])
    tol = max(1e-10, 2.3e-15 * (1 + lam * m))
    assert np.all(np.linalg.norm(got - ref, axis=0) <= 2 * tol * np.linalg.norm(b, axis=0))


def test_odd_last_iteration_returns_the_last_iterate():
    dev = device()
    nv, edges = _case("path")
    A, off, adj = _graph(nv, edges)
    M = np.eye(nv) + 20.0 * (np.diag(A.sum(1)) - A)
    b = np.random.default_rng(1).normal(size=(nv, 3))
    s = B.Smooth(torch.from_numpy(off).to(dev), torch.from_numpy(adj).to(dev), 20.0)
    bt = torch.from_numpy(b).to(dev)
    res = []
    for k in (1, 2, 7, 8):
        x = torch.zeros(nv, 3, dtype=torch.float64, device=dev)
        with pytest.raises(B.DTError):
            s.solve(bt, x, max_iters=k)
        assert s.iters == k
        r = np.linalg.norm(b - M @ x.cpu().numpy(), axis=0) / np.linalg.norm(b, axis=0)
        assert abs(r.max() - s.resid) <= 1e-12
        res.append(r.max())
    assert res[0] > res[1] > res[2] > res[3]
