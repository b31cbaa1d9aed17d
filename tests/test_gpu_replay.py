"""The backward of a checkpointed trace takes the hits of the generations on the
tape from the triangles noted there.  Against the trace that stores everything:
the same records go into the same sums, so the gradients agree to the order of
the float sums, at ray counts around a wave and a block, on one triangle, and
when the backward runs twice on one tape."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import DV_ORDER_TOL, device

pytestmark = pytest.mark.gpu


def _mesh(kind):
    if kind == "triangle":
        return np.float32([[-1, -1, 0], [1, -1, 0.1], [0, 1, 0]]), np.int32([[0, 1, 2]])
    V, F = synth.displaced_torus(seed=4, nu=24, nv=13)
    return np.asarray(V, np.float32), np.asarray(F, np.int32)


def _grads(scene, rays, env, depth, stride, g, times=1):
    p = B.Params(max_depth=depth, checkpoint_stride=stride)
    buf = B.Buffers(p, rays, scene.mesh, tape=True)
    rgb = B.dt_trace_forward(scene, rays, p, buf)[0]
    for _ in range(times):
        dV, de, ds = B.dt_trace_backward(scene, rays, p, buf, g)
    return rgb.clone(), dV.cpu().double(), float(de), ds.cpu().double()


@pytest.mark.parametrize("kind,n,depth,stride", [
    ("triangle", 65, 2, 2), ("torus", 1, 5, 2), ("torus", 63, 5, 3), ("torus", 257, 6, 2), ("torus", 2049, 4, 4),
    ("torus", 4096, 4, 9)])
def test_replayed_generations(kind, n, depth, stride):
    dev = device()
    V, F = _mesh(kind)
    mesh = B.Mesh(torch.from_numpy(V).to(dev), torch.from_numpy(F).to(dev))
    env = B.Env(torch.from_numpy(synth.env_equirect(64, 32, seed=3)).to(dev))
    scene = B.Scene(mesh, torch.tensor([1.4], device=dev), torch.tensor([0.3, 0.2, 0.1], device=dev), env)
    rng = np.random.default_rng(n)
    o = rng.normal(size=(n, 3))
    o = 3.0 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.9, 0.9, (n, 3)) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    o, d = (torch.from_numpy(x.astype(np.float32)).to(dev) for x in (o, d))
    rays = B.Rays(o=o, d=d)
    g = torch.from_numpy(rng.normal(size=(n, 3)).astype(np.float32)).to(dev)
    rgb1, dV1, de1, ds1 = _grads(scene, rays, env, depth, 1, g)
    rgb2, dV2, de2, ds2 = _grads(scene, rays, env, depth, stride, g, times=2)
    # a pixel sums at most 2^depth paths, in any order
    assert (rgb1 - rgb2).abs().max() <= 2**depth * 2**-23 * rgb1.abs().max()
    assert torch.linalg.norm(dV1 - dV2) <= DV_ORDER_TOL * torch.linalg.norm(dV1) + 1e-9
    assert abs(de1 - de2) <= 1e-6 * abs(de1) + 1e-9
    assert torch.linalg.norm(ds1 - ds2) <= 1e-6 * torch.linalg.norm(ds1) + 1e-9
