"""The solve's workspace: three float64 vectors and the partial sums, whichever
recurrence runs, and nothing written past it."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from tests.gpu_helpers import device
from tests.test_gpu_smooth_rows import _case, _graph


def _room(nv):
    """Three vectors of [nv, 3], six partial sums and a degree per block of 256, eight totals."""
    blocks = -(-nv // 256)
    return sum(-(-n // 256) * 256 for n in (24 * nv, 24 * nv, 24 * nv, 48 * blocks, 4 * blocks, 64))


@pytest.mark.parametrize("nv", [1, 2, 3, 255, 256, 257, 642, 154608, (1 << 28) - 1])
def test_workspace_size(nv):
    n = C.c_size_t()
    B._check(B.load().dt_smooth_bytes(nv, C.byref(n)))
    assert n.value <= _room(nv)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["single", "star", "degree9", "path"])
@pytest.mark.parametrize("lam", [3.0, 1e4])   # on the iterates, and with the residual carried
def test_solve_in_it(kind, lam):
    dev = device()
    nv, edges = _case(kind)
    A, off, adj = _graph(nv, edges)
    M = np.eye(nv) + lam * (np.diag(A.sum(1)) - A)
    b = np.random.default_rng(nv).normal(size=(nv, 3))
    adj = adj if len(adj) else np.zeros(1, np.int32)
    s = B.Smooth(torch.from_numpy(off).to(dev), torch.from_numpy(adj).to(dev), lam)
    room = _room(nv)
    around = torch.full((room + 4096,), 0xA5, dtype=torch.uint8, device=dev)
    s.ws = around[:room]
    x = torch.zeros(nv, 3, dtype=torch.float64, device=dev)
    s.solve(torch.from_numpy(b).to(dev), x, max_iters=20000)
    assert (around[room:] == 0xA5).all()
    # the residual met the tolerance of 1e-10 a column; its own rounding is 20 u (1 + lam m),
    # m at most twice the largest degree
    r = np.linalg.norm(b - M @ x.cpu().numpy(), axis=0) / np.linalg.norm(b, axis=0)
    assert r.max() <= 2 * max(1e-10, 2.3e-15 * (1 + 2 * lam * A.sum(1).max()))
