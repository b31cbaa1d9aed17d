"""The outline gradient's cut into waves, below and above 2^19 edge slots and over
numbers of cameras that its groups do not divide: several views in one call
give the sum of one view a call, and count the same outline points.  On
separate triangles, whose every edge is on the outline, eight views cost about
eight times one."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


def _soup(n, seed):
    rng = np.random.default_rng(seed)
    V = (rng.uniform(-1, 1, (n, 1, 3)) + rng.normal(0, 0.02, (n, 3, 3))).reshape(-1, 3)
    return V, np.arange(3 * n).reshape(-1, 3)


def _mesh(V, F, dev):
    return B.Mesh(torch.from_numpy(V.astype(np.float32)).to(dev), torch.from_numpy(F.astype(np.int32)).to(dev))


@pytest.mark.parametrize("views", [1, 2, 3, 5, 16])
@pytest.mark.parametrize("faces", [21, 22, 2000, (1 << 19) // 3, (1 << 19) // 3 + 1])   # 63, 66, ... slots
def test_views_add_up(faces, views):
    dev = device()
    mesh = _mesh(*_soup(faces, seed=views), dev)
    cams = [synth.look_at_camera(e, 24, 20) for e in synth.views_on_sphere(views, 3.0, seed=views)]
    g = np.random.default_rng(faces).normal(size=(views, 24 * 20)).astype(np.float32)
    mg = B.MaskGrad(mesh)
    dV = mg(mesh, B.Rays(cameras=cams), torch.from_numpy(g.reshape(-1)).to(dev)).cpu().numpy()
    counts = mg.counts.clone()
    one, size, parts = 0.0, 0.0, torch.zeros_like(counts)
    for c, gc in zip(cams, g):
        d = mg(mesh, B.Rays(cameras=[c]), torch.from_numpy(gc).to(dev)).cpu().numpy().astype(np.float64)
        one, size, parts = one + d, size + np.abs(d), parts + mg.counts
    assert counts[0] > 0 and torch.equal(counts, parts)
    # the terms are the same numbers; a vertex adds at most some 40 points of its two
    # edges from each view, in any order
    assert np.all(np.abs(dV - one) <= 40 * views * 2.0 ** -24 * np.maximum(size, 1e-30) * 8)


def test_separate_triangles():
    dev = device()
    mesh = _mesh(*_soup(20000, seed=0), dev)
    ms = []
    for views in (1, 8):
        rays = B.Rays(cameras=[synth.look_at_camera(e, 512, 512) for e in synth.views_on_sphere(views, 3.0, seed=4)])
        g = torch.randn(rays.n_pixels, device=dev, generator=torch.Generator(dev).manual_seed(1))
        mg, t = B.MaskGrad(mesh), []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            mg(mesh, rays, g)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(min(t))
    print(f"one view {ms[0]:.2f} ms, eight {ms[1]:.2f}", flush=True)
    # 28.9 ms and 256 slots a wave for eight, 3.6 now; one thread per edge and camera 14.0
    assert ms[1] <= 12.0
