"""Coverage masks of images narrower or lower than a tile of 8 x 8 pixels, alone
and several to a call: each pixel as the tracer's camera ray finds it; and the
longest strip, which a launch of 8 x 8 tiles could not hold."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 500), (2, 333), (3, 101), (4, 64), (5, 70), (7, 9), (500, 1), (333, 2), (101, 3), (64, 4),
         (70, 5), (8, 8), (9, 7), (9, 9), (63, 65)]


def _mesh(V, F, dev):
    return B.Mesh(torch.from_numpy(V.astype(np.float32)).to(dev), torch.from_numpy(F.astype(np.int32)).to(dev))


def _check(cams, dev):
    mesh = _mesh(*synth.icosphere(2), dev)
    env = B.Env(torch.ones(2, 4, 3, device=dev))
    scene = B.Scene(mesh, torch.tensor([1.4], device=dev), torch.zeros(3, device=dev), env)
    rays, p = B.Rays(cameras=cams), B.Params(max_depth=0)
    _, _, fl = B.dt_trace_forward(scene, rays, p, B.Buffers(p, rays, mesh, tape=False))
    hit = (fl & B.FLAG_TRUNC) != 0
    assert hit.any()
    assert torch.equal(B.dt_mask_forward(mesh, rays) != 0, hit)


@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_narrow_image(size):
    _check([synth.look_at_camera(np.array([0.9, 2.4, 1.3]), *size)], device())


def test_narrow_images_in_one_call():
    eyes = synth.views_on_sphere(len(SIZES), 3.0, seed=1)
    _check([synth.look_at_camera(e, *s) for e, s in zip(eyes, SIZES)], device())


def test_longest_strip():
    """2^29 + 8 rows of one pixel, seen from inside the object."""
    dev = device()
    mesh = _mesh(*synth.icosphere(1), dev)
    cam = synth.look_at_camera(np.array([0.0, 0.1, 0.3]), 1, (1 << 29) + 8)
    mask = B.dt_mask_forward(mesh, B.Rays(cameras=[cam]))
    assert mask.numel() == (1 << 29) + 8 and bool((mask == 1.0).all())
