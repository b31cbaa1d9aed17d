"""The scatter of the field's gradient where waves add to few cells: sums that run
over several of a wave's groups go out once, and a backward through coarse
planes takes about as long as through fine ones."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import device, icosphere_pair
from tests.test_gpu_field import HI, LO, _grad_check, _with_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,res", [
    ((2, 2, 2), 9),     # every record of a wave in one grid cell, planes' over a few groups
    ((9, 8, 7), 2),     # one cell a plane
    ((3, 2, 2), 3),     # two grid cells: a boundary anywhere in the order
    ((2, 4, 3), 4),
])
def test_few_cells(n, res):
    P = _with_field(icosphere_pair(sigma=(0.5, 0.2, 0.1), res=48), seed=31, samples=3, n=n, res=res, box=(LO, HI))
    _grad_check(P, seed=32, label=f"field {n} planes {res}")


def test_coarse_planes_take_no_longer():
    dev = device()
    V, F = synth.displaced_torus(seed=1, nu=160, nv=80)
    mesh = B.Mesh(torch.from_numpy(V.astype(np.float32)).to(dev), torch.from_numpy(F.astype(np.int32)).to(dev))
    rays = B.Rays(cameras=[synth.look_at_camera(e, 400, 400) for e in synth.views_on_sphere(2, 3.0, seed=2)])
    p = B.Params(max_depth=5, queue_capacity=2 * rays.n_rays)
    buf = B.Buffers(p, rays, mesh, tape=True)
    gen = torch.Generator(dev).manual_seed(1)
    g = torch.randn(rays.n_pixels, 3, device=dev, generator=gen)
    ms = []
    for res in (33, 2):
        fld = B.Field(torch.randn(33, 33, 33, 4, device=dev, generator=gen) - 1.0,
                      0.3 * torch.randn(3, res, res, 4, device=dev, generator=gen), V.min(0) - 0.3, V.max(0) + 0.3, 8)
        sc = B.Scene(mesh, torch.tensor([1.45], device=dev), torch.full((3,), 0.3, device=dev),
                     B.Env(torch.ones(4, 8, 3, device=dev)), field=fld)
        B.dt_trace_forward(sc, rays, p, buf)
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.dt_trace_backward(sc, rays, p, buf, g)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(min(t))
    print(f"planes of 33 x 33: {ms[0]:.2f} ms, of 2 x 2: {ms[1]:.2f}", flush=True)
    assert ms[1] <= 2.0 * ms[0]
