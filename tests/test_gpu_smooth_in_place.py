"""The solve where the solution's array is, or overlaps, the right-hand side's:
x holds the starting guess on entry, so b = x starts from b."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from tests.gpu_helpers import device
from tests.test_gpu_smooth_rows import _case, _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["star", "degree9", "path"])
@pytest.mark.parametrize("shift", [0, 1, -3])   # x starts that many vertices after b
def test_in_place(kind, shift):
    dev = device()
    nv, edges = _case(kind)
    A, off, adj = _graph(nv, edges)
    lam = 3.0
    M = np.eye(nv) + lam * (np.diag(A.sum(1)) - A)
    s = B.Smooth(torch.from_numpy(off).to(dev), torch.from_numpy(adj).to(dev), lam)
    both = torch.from_numpy(np.random.default_rng(nv).normal(size=(nv + 8, 3))).to(dev)
    b, x = both[4:4 + nv], both[4 + shift:4 + shift + nv]
    want = b.cpu().numpy().copy()
    s.solve(b, x)
    # |error| <= |residual| <= 1e-10 |b| a column (the smallest eigenvalue is 1); the
    # reference's and the residual's own rounding stay far below that at this lambda
    err = np.linalg.norm(x.cpu().numpy() - np.linalg.solve(M, want), axis=0)
    assert np.all(err <= 2e-10 * np.linalg.norm(want, axis=0))
