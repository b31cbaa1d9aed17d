"""The field's ray adjoint behind an opaque wall: camera segments that end on a
surface far past the point where the transmittance vanishes, with steep
densities there.  What lies behind contributes nothing to the gradient of the
segment's end, and its rounding must not either: each ray's dL/dt against the
FP64 derivative of the same sums, at a multiple of the FP32 rounding of the
terms that the transmittance leaves."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu

N, NODES = 1024, 9


def _feature(grid, x):
    """Trilinear value of nodes over [-1, 1]^3 (grid[z, y, x]) at x [N, 3], float64."""
    n = grid.shape[0]
    u = ((x + 1.0) * ((n - 1) / 2.0)).clamp(0.0, n - 1.0)
    i = u.detach().floor().clamp(max=n - 2).long()
    f = u - i
    out = 0.0
    for k in range(8):
        c = (k & 1, (k >> 1) & 1, k >> 2)
        w = [f[:, a] if c[a] else 1.0 - f[:, a] for a in range(3)]
        out = out + (w[0] * w[1] * w[2])[:, None] * grid[i[:, 2] + c[2], i[:, 1] + c[1], i[:, 0] + c[0]]
    return out


def _reference(grid, o, d, t, Lb, S):
    """dL/dt of the emission's sum over S midpoints of [0, t], and the sum of the
    magnitudes of its terms, each with the transmittance in front of it."""
    ts = t.clone().requires_grad_(True)
    h = ts / S
    T, C, rows = torch.ones_like(t), 0.0, []
    for k in range(S):
        x = o + d * (h * (k + 0.5))[:, None]
        f = _feature(grid, x)
        sig = torch.nn.functional.softplus(f[:, 0], threshold=35.0)
        a = torch.exp(-sig * h)
        w = T * (1.0 - a)
        C = C + f[:, 1:] * w[:, None]
        T = T * a
        slope = torch.stack([torch.autograd.grad(f[:, c].sum(), x, retain_graph=True)[0].mul(d).sum(1)
                             for c in range(4)], 1)
        rows.append((f.detach(), sig.detach(), w.detach(), T.detach(), slope))
    ref, = torch.autograd.grad((C * Lb).sum(), ts)
    A, behind = torch.zeros_like(t), torch.zeros(len(t), 3, dtype=t.dtype)
    for k in range(S - 1, -1, -1):
        f, sig, w, T, slope = rows[k]
        g = (Lb.abs() * (f[:, 1:].abs() * T[:, None] + behind)).sum(1)
        A += sig * g + (k + 0.5) * (slope[:, 0].abs() * h.detach() * torch.sigmoid(f[:, 0]) * g
                                    + (slope[:, 1:].abs() * Lb.abs()).sum(1) * w)
        behind += f[:, 1:].abs() * w[:, None]
    return ref.numpy(), (A / S).numpy()


@pytest.mark.parametrize("samples", [16, 64, 128])
def test_segment_end_behind_a_wall(samples):
    dev = device()
    rng = np.random.default_rng(samples)
    grid = np.empty((NODES, NODES, NODES, 4))
    wall = np.array([1, 1, 1, 20, 100, 1e4, 1e4, 1e4, 1e4])
    grid[..., 0] = wall[:, None, None] * rng.uniform(0.5, 1.5, (NODES,) * 3)
    grid[..., 1:] = rng.uniform(0, 1, (NODES, NODES, NODES, 3))
    grid = grid.astype(np.float32)
    # the whole segment lies in the field's box: it starts and ends there
    o = rng.uniform(-0.5, 0.5, (N, 3))
    o[:, 2] = -0.95
    d = np.array([0.0, 0.0, 1.0]) + rng.uniform(-0.2, 0.2, (N, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    o, d = o.astype(np.float32), d.astype(np.float32)
    # one triangle per ray, across its way at a distance of 1.5 to 1.8 inside the
    # box; the rays' own lines do not meet each other's triangles first (checked
    # below by the hit's triangle)
    t = rng.uniform(1.5, 1.8, N)
    hit = o + d * t[:, None]
    assert np.abs(hit).max() < 1.0
    side = np.cross(d, [1.0, 0.0, 0.0])
    side /= np.linalg.norm(side, axis=1, keepdims=True)
    up = np.cross(side, d)
    r = 0.004
    V = np.stack([hit + r * (-side - up), hit + r * (side - up), hit + r * up * 2], 1).reshape(-1, 3).astype(np.float32)
    F = np.arange(3 * N, dtype=np.int32).reshape(-1, 3)
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    mesh = B.Mesh(dv(V), dv(F))
    fld = B.Field(dv(grid), torch.zeros(3, 2, 2, 4, device=dev), (-1.0,) * 3, (1.0,) * 3, samples)
    scene = B.Scene(mesh, torch.tensor([1.5], device=dev), torch.zeros(3, device=dev),
                    B.Env(torch.ones(2, 4, 3, device=dev)), field=fld)
    rays, p = B.Rays(dv(o), dv(d)), B.Params(max_depth=0)
    tri, _, _ = B.dt_intersect(scene, dv(o), dv(d))
    own = tri.cpu().numpy() == np.arange(N)
    assert own.mean() > 0.9
    buf = B.Buffers(p, rays, mesh, tape=True)
    rgb, _, _ = B.dt_trace_forward(scene, rays, p, buf)
    assert (rgb[torch.from_numpy(own).to(dev)] > 0).all()   # met from outside: the field's emission
    Lb = rng.normal(size=(N, 3)).astype(np.float32) * own[:, None]
    dV, _, _ = B.dt_trace_backward(scene, rays, p, buf, dv(Lb.astype(np.float32)))
    # t depends on its triangle's plane alone, d t / d(common shift s) = n . s / n . d,
    # so the three vertices' gradients add up to dL/dt n / (n . d)
    got = (dV.cpu().numpy().astype(np.float64).reshape(N, 3, 3).sum(1) * d).sum(1)
    V64, o64, d64 = V.astype(np.float64).reshape(N, 3, 3), o.astype(np.float64), d.astype(np.float64)
    n = np.cross(V64[:, 1] - V64[:, 0], V64[:, 2] - V64[:, 0])
    t64 = ((V64[:, 0] - o64) * n).sum(1) / (d64 * n).sum(1)
    T = lambda a: torch.from_numpy(np.asarray(a, np.float64))  # noqa: E731
    ref, A = _reference(T(grid), T(o64), T(d64), T(t64), T(Lb), samples)
    # In units u = 2^-24 of a term: 24 for the taps of a sample's density times the
    # optical depth of 17 after which nothing is left, 32 for a sample's place
    # in the grid times the densities' differences passed on the way (at most
    # 19 and 80 over cells 0.25 long), some 10 for the products of a term and
    # its sum, and 50 for the triangle's part: below 2,048 together
    err = np.abs(got - ref)[own] / (A[own] * 2.0 ** -24)
    print(f"S={samples}: error in units of rounding: median {np.median(err):.1f}, largest {err.max():.1f}", flush=True)
    assert err.max() <= 2048.0
