"""A mesh with a small piece far away from the rest: rays that pass the rest find
the same hits and cost about what they cost without the piece."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


def _render(V, F, dev):
    """Path signatures of two views, and the forward render's time in ms (the
    least of some runs)."""
    mesh = B.Mesh(torch.from_numpy(V.astype(np.float32)).to(dev), torch.from_numpy(F.astype(np.int32)).to(dev))
    env = B.Env(torch.from_numpy(synth.env_equirect(64, 32, seed=1)).float().to(dev))
    scene = B.Scene(mesh, torch.tensor([1.45], device=dev), torch.full((3,), 0.3, device=dev), env)
    rays = B.Rays(cameras=[synth.look_at_camera(e, 400, 400) for e in synth.views_on_sphere(2, 3.0, seed=2)])
    p = B.Params(max_depth=6, queue_capacity=2 * rays.n_rays)
    buf = B.Buffers(p, rays, mesh, tape=False)
    sig = torch.zeros(rays.n_pixels, dtype=torch.int64, device=dev)
    ms = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        B.dt_trace_forward(scene, rays, p, buf, path_sig=sig)
        b.record()
        b.synchronize()
        ms.append(a.elapsed_time(b))
    return sig.cpu().numpy(), min(ms)


def _with_piece(V, F, away):
    tet = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]])
    tf = np.array([[0, 2, 1], [0, 1, 3], [1, 2, 3], [0, 3, 2]])
    return (np.concatenate([V, 0.01 * tet + away * np.array([1.0, 0.9, -0.8])]),
            np.concatenate([F, tf + len(V)]))


def _compare(nu, away, most):
    dev = device()
    V, F = synth.displaced_torus(seed=1, nu=nu, nv=nu // 2)
    sig0, ms0 = _render(V, F, dev)
    sig1, ms1 = _render(*_with_piece(V, F, away), dev)
    print(f"{len(F)} faces: {ms0:.2f} ms, with the piece {away:g} away {ms1:.2f}", flush=True)
    # the piece covers no pixel's centre and takes no secondary ray of a view
    assert (sig0 != sig1).sum() <= 2
    assert ms1 <= most * ms0


@pytest.mark.parametrize("away", [1e3, 1e4])
def test_boxes_stay_tight(away):
    """What the boxes are widened by against rounding follows the node, not the
    whole tree (which measured 1.8 and 9.2 times as long here; the nodes' own
    bounds 1.4 and 1.6, the rest of it from the Morton grid's coarser cells)."""
    _compare(320, away, 3.0)


@pytest.mark.parametrize("away", [1e3, 1e4])
def test_large_mesh_keeps_its_order(away):
    """Above 2^20 faces the Morton grid's cells are fine enough for detail in a
    small part of the mesh's box (keys of 32 bits measured 2.5 and 4.1 times as
    long here, of 63 bits 1.0)."""
    _compare(1100, away, 2.0)
