"""The work that users of this framework have it do, as cases to be timed.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (mesh, cameras, environment, optimiser targets, a resident server),
`run` is one pass through the public entry points, `work` the bytes and
operations a pass cannot do without, and `exact` the same outputs in 64 bits
from plain torch where the size allows it.

Kinds:
  batch   the paper's training batch: a few thousand explicit rays, tree
          rebuilt, forward with a tape, backward
  view    one image, forward only (inference), flags and truncated weight too
  step    a training step on whole images through `autograd.render`,
          `render_grid` (absorption grid) or `render_mlp` (network trained)
  field   a training step with the volumetric field outside the object, the
          field's and the map's texel gradients written
  shell   a thin hollow wall: many trapped rays, deep, recomputed from a
          partial tape, lit by a network
  serve   a burst of requests on resident scenes through the server
  mask    coverage of the views and its outline gradient
  solve   vertices from the reparameterised unknowns, (I + lambda L) V = u
  build   tree and normals of a changed mesh, and picks through the new tree
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2603_00413_amd import autograd as A
from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from paper_2603_00413_amd import train as T
from paper_2603_00413_amd.serve import Request, Server

DEV = "cuda:0"


def listed():
    return [
        # the paper's ray batch (5,000 rays, at most 4 bounces) on a mesh of
        # ordinary size: launches and latency
        dict(name="batch-5k", kind="batch", rays=5000, nu=320, nv=160, depth=4),
        # the smallest render: a preview of the 1,280-face icosphere
        dict(name="view-icosphere-64", kind="view", mesh="icosphere", nu=3, nv=0, width=64, height=64, depth=4),
        # one image of a ragged size at the inference depth
        dict(name="view-torus-801x601", kind="view", mesh="torus", nu=320, nv=160, width=801, height=601, depth=8),
        # the benchmark's training step: 8 whole views, constant absorption
        dict(name="step-torus", kind="step", mesh="torus", nu=320, nv=160, views=8, width=512, height=512, depth=6,
             env="map", grid=0, samples=0),
        # the training shape: ~300k faces, 8 views of 800 x 800, the lighting
        # network trained with the mesh
        dict(name="step-sdf-mlp", kind="step", mesh="sdf", nu=222, nv=3, views=8, width=800, height=800, depth=6,
             env="mlp", grid=0, samples=0),
        # an absorbing interior that varies in space, its grid trained
        dict(name="step-grid", kind="step", mesh="torus", nu=320, nv=160, views=8, width=512, height=512, depth=6,
             env="map", grid=32, samples=16),
        # a scene inside a volumetric environment, field and map trained
        dict(name="step-field", kind="field", nu=320, nv=160, views=8, width=512, height=512, depth=6, grid=32,
             res=64, samples=8),
        # the largest: a 2M-face thin wall at 1024 x 1024, depth 8 (some 60M
        # segments, most of them trapped in the wall), a wide network, every
        # second generation on the tape
        dict(name="shell-2m", kind="shell", nu=1024, nv=512, width=1024, height=1024, depth=8, stride=2, layers=4,
             hidden=128),
        # a burst on four resident scenes, images of 128 to 1024 pixels a side
        dict(name="serve-burst", kind="serve", requests=20, scale=1.0),
        # the periodic silhouette term of the same 8 views
        dict(name="mask-torus", kind="mask", nu=320, nv=160, views=8, width=512, height=512),
        # the mesh optimiser's solve at the training shape
        dict(name="solve-sdf", kind="solve", mesh="sdf", nu=222, nv=3, lam=20.0),
        # the acceleration data of a large mesh after its vertices moved
        dict(name="build-2m", kind="build", nu=1448, nv=724, picks=4096),
    ]


def draw(rng):
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def torus(lo, hi):
        nu = span(lo, hi)
        return dict(nu=nu, nv=max(12, nu // 2 + rng.randint(-5, 5)))

    kind = rng.choice(["batch", "batch", "view", "view", "step", "step", "step", "field", "shell", "serve", "mask",
                       "solve", "build"])
    if kind == "batch":
        return dict(kind=kind, rays=span(500, 20000), depth=rng.randint(2, 6), **torus(48, 320))
    if kind == "view":
        return dict(kind=kind, mesh="torus", width=span(40, 1100), height=span(40, 1100), depth=rng.randint(4, 8),
                    **torus(32, 512))
    if kind == "step":
        form = rng.choice(["map", "mlp", "grid"])
        return dict(kind=kind, mesh="torus", views=rng.randint(1, 8), width=span(80, 600), height=span(80, 600),
                    depth=rng.randint(3, 6), env="mlp" if form == "mlp" else "map",
                    grid=rng.randint(9, 48) if form == "grid" else 0,
                    samples=rng.randint(4, 24) if form == "grid" else 0, **torus(64, 400))
    if kind == "field":
        return dict(kind=kind, views=rng.randint(1, 6), width=span(80, 512), height=span(80, 512),
                    depth=rng.randint(3, 6), grid=rng.randint(9, 48), res=rng.randint(17, 96),
                    samples=rng.randint(4, 16), **torus(64, 400))
    if kind == "shell":
        return dict(kind=kind, width=span(100, 1000), height=span(100, 1000), depth=rng.randint(5, 8),
                    stride=rng.randint(2, 3), layers=rng.randint(2, 4), hidden=rng.choice([64, 128]),
                    **torus(128, 1024))
    if kind == "serve":
        return dict(kind=kind, requests=rng.randint(3, 20), scale=rng.choice([0.25, 0.5, 1.0]))
    if kind == "mask":
        return dict(kind=kind, views=rng.randint(1, 8), width=span(64, 800), height=span(64, 512), **torus(64, 400))
    if kind == "solve":
        return dict(kind=kind, mesh="torus", lam=rng.uniform(5.0, 60.0), **torus(64, 560))
    return dict(kind=kind, picks=span(500, 20000), **torus(32, 1400))


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=2)
def _sdf(res, seed):
    return synth.sdf_union_mesh(seed, res)


def _turn(rng):
    """A random rotation matrix."""
    q = rng.normal(size=4)
    w, x, y, z = q / np.linalg.norm(q)
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                     [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                     [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])


def _mesh(case, seed):
    """Vertices [nv, 3] float32 and faces [nf, 3] int32 (numpy) of the case's mesh."""
    rng = np.random.default_rng([seed, 1])
    kind = case.get("mesh", "torus")
    if kind == "icosphere":
        V, F = synth.icosphere(case["nu"])
        V = V @ _turn(rng).T
    elif kind == "sdf":
        V, F = _sdf(case["nu"], case["nv"])
        V = V @ _turn(rng).T
    else:
        V, F = synth.displaced_torus(seed=seed, nu=case["nu"], nv=case["nv"])
        if case["kind"] == "shell":
            # a hollow wall: the same surface 0.02 further in, facing inwards
            Vi, Fi = synth.displaced_torus(seed=seed, r=0.28, nu=case["nu"], nv=case["nv"])
            F = np.concatenate([F, Fi[:, ::-1] + len(V)])
            V = np.concatenate([V, Vi])
    return V.astype(np.float32), np.ascontiguousarray(F, dtype=np.int32)


def _faces(case):
    """(vertices, faces) of the case's mesh, by count."""
    kind = case.get("mesh", "torus")
    if kind == "icosphere":
        return 10 * 4 ** case["nu"] + 2, 20 * 4 ** case["nu"]
    if kind == "sdf":
        nf = 6.28 * case["nu"] ** 2
        return nf / 2, nf
    n = case["nu"] * case["nv"] * (2 if case["kind"] == "shell" else 1)
    return n, 2 * n


def _cameras(case, seed):
    eyes = synth.views_on_sphere(case.get("views", 1), 3.0, seed=seed)
    return [synth.look_at_camera(e, case["width"], case["height"]) for e in eyes]


def _dev(a, dtype=None):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def _material(seed):
    rng = np.random.default_rng([seed, 2])
    return (torch.tensor([rng.uniform(1.37, 1.6)], dtype=torch.float32, device=DEV),
            torch.tensor(rng.uniform(0.1, 0.5, 3), dtype=torch.float32, device=DEV))


def _target(n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return 0.2 + 0.5 * torch.rand(n, 3, generator=g, device=DEV)


def _batch_rays(n, seed):
    """n rays through random points of 8 views' image planes."""
    rng = np.random.default_rng([seed, 3])
    eye = synth.views_on_sphere(8, 3.0, seed=seed)[rng.integers(0, 8, n)]
    f = -eye / np.linalg.norm(eye, axis=1, keepdims=True)
    r = np.cross(f, [0.0, 1.0, 0.0])
    r /= np.linalg.norm(r, axis=1, keepdims=True)
    u = np.cross(r, f)
    p = rng.uniform(-1, 1, (n, 2)) * math.tan(math.radians(20.0))
    d = f + r * p[:, :1] + u * p[:, 1:]
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return eye.astype(np.float32), d.astype(np.float32)


def _mlp(seed, layers, hidden, train):
    Ws, Bs = synth.env_mlp_weights(seed, n_layers=layers, width=hidden)
    return Ws, Bs, B.Env.mlp(Ws, Bs, 6, DEV, want_grad=train)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return _prepare_serve(case, seed)
    Vn, Fn = _mesh(case, seed)
    V, F = _dev(Vn), _dev(Fn)
    s = dict(kind=kind, V=V, F=F)
    if kind == "solve":
        s["ls"] = T.LargeSteps(len(Vn), F, case["lam"])
        s["u"] = s["ls"].to_u(V)
        return s
    if kind == "build":
        s["mesh"] = B.Mesh(V, F)
        s["o"], s["d"] = (_dev(a) for a in _batch_rays(case["picks"], seed))
        env = B.Env(_dev(synth.env_equirect(16, 8, seed=seed)))
        s["scene"] = B.Scene(s["mesh"], *_material(seed), env)
        return s
    s["ior"], s["sigma"] = _material(seed)
    if kind == "mask":
        s["V"] = V.requires_grad_(True)
        s["tracer"] = A.Tracer(F, B.Env(_dev(synth.env_equirect(16, 8, seed=seed))), _cameras(case, seed))
        s["target"] = _target(s["tracer"].rays.n_pixels, seed)[:, 0].contiguous()
        return s
    if kind == "step":
        if case["env"] == "mlp":
            Ws, Bs, env = _mlp(seed, 3, 64, True)
            s["w"], s["b"] = (_dev(np.concatenate([x.reshape(-1) for x in p])).requires_grad_(True) for p in (Ws, Bs))
        else:
            env = B.Env(_dev(synth.env_equirect(512, 256, seed=seed)))
        s["tracer"] = A.Tracer(F, env, _cameras(case, seed), max_depth=case["depth"])
        s["target"] = _target(s["tracer"].rays.n_pixels, seed)
        for k in ("V", "ior", "sigma"):
            s[k].requires_grad_(True)
        if case["grid"]:
            n = case["grid"]
            mu = np.random.default_rng([seed, 4]).uniform(0.1, 0.5, (n, n, n, 3))
            s["mu"] = _dev(mu, torch.float32).requires_grad_(True)
            s["lo"], s["hi"], s["samples"] = Vn.min(0) - 0.01, Vn.max(0) + 0.01, case["samples"]
        return s
    # the remaining kinds call the library's own entry points
    s["mesh"] = B.Mesh(V, F)
    field = None
    if kind == "shell":
        env = _mlp(seed, case["layers"], case["hidden"], False)[2]
    else:
        env = B.Env(_dev(synth.env_equirect(64 if kind == "view" and case["mesh"] == "icosphere" else 512,
                                            32 if kind == "view" and case["mesh"] == "icosphere" else 256,
                                            seed=seed)), want_grad=kind == "field")
    if kind == "field":
        rng = np.random.default_rng([seed, 5])
        n, r = case["grid"], case["res"]
        grid = np.concatenate([rng.normal(-1.5, 0.6, (n, n, n, 1)), rng.uniform(0, 0.5, (n, n, n, 3))], -1)
        planes = np.concatenate([rng.normal(0, 0.4, (3, r, r, 1)), rng.uniform(-0.1, 0.2, (3, r, r, 3))], -1)
        field = B.Field(_dev(grid, torch.float32), _dev(planes, torch.float32), Vn.min(0) - 0.3, Vn.max(0) + 0.3,
                        case["samples"])
    s["scene"] = B.Scene(s["mesh"], s["ior"], s["sigma"], env, field=field)
    if kind == "batch":
        s["rays"] = B.Rays(*(_dev(a) for a in _batch_rays(case["rays"], seed)))
    else:
        s["rays"] = B.Rays(cameras=_cameras(case, seed))
    # room for the trapped rays of a thin wall; twice the camera rays elsewhere
    cap = (40 if kind == "shell" else 2) * s["rays"].n_rays
    s["params"] = B.Params(max_depth=case["depth"], queue_capacity=cap, checkpoint_stride=case.get("stride", 1))
    s["buf"] = B.Buffers(s["params"], s["rays"], s["mesh"], tape=kind != "view")
    s["target"] = _target(s["rays"].n_pixels, seed)
    return s


SERVE_FACES = ((224, 112), (384, 196), (556, 270), (714, 350))   # ~50k, 150k, 300k, 500k faces


def _serve_requests(case, seed):
    """(scene, environment, pixels a side, depth) of each request."""
    rng = np.random.default_rng([6, case["requests"]])
    sides = [128, 256, 512, 1024]
    rows = []
    for i in range(case["requests"]):
        res = int(case["scale"] * sides[i % 4])
        relight = None if rng.uniform() < 0.7 else 4 + int(rng.integers(0, 4))
        rows.append((int(rng.integers(0, 4)), relight, res, int(rng.integers(4, 9))))
    return rows


def _prepare_serve(case, seed):
    rng = np.random.default_rng([seed, 7])
    srv = Server(DEV, queue_capacity=8 << 20, pixel_pool=8 << 20)
    for k, (nu, nv) in enumerate(SERVE_FACES):
        V, F = synth.displaced_torus(seed=seed + k, nu=nu, nv=nv)
        srv.add_scene(V, F, float(rng.uniform(1.37, 1.6)), tuple(rng.uniform(0.05, 0.5, 3)),
                      synth.env_equirect(512, 256, seed=seed + 100 + k))
    for k in range(2):
        srv.add_env(synth.env_equirect(512, 256, seed=seed + 200 + k))
    for k, (layers, width) in enumerate([(3, 64), (2, 128)]):
        srv.add_env(_mlp(seed + 210 + k, layers, width, False)[2])
    rows = _serve_requests(case, seed)
    eyes = synth.views_on_sphere(len(rows), 3.0, seed=seed)
    reqs = [Request(i, sc, synth.look_at_camera(eyes[i], res, res), dep, env)
            for i, (sc, env, res, dep) in enumerate(rows)]
    return dict(kind="serve", server=srv, requests=reqs)


# ------------------------------------------------------------------ one pass
def run(s):
    kind = s["kind"]
    if kind == "serve":
        return [[r.image, r.flags, r.sig.view(np.int64)] for r in s["server"].run(s["requests"])]
    if kind == "solve":
        return s["ls"].to_v(s["u"], slot=None)
    if kind == "build":
        s["mesh"].build()
        tri, t, b = B.dt_intersect(s["scene"], s["o"], s["d"])
        return dict(normals=s["mesh"].vertex_normals(), tri=tri, t=t, b=b)
    if kind == "mask":
        m = A.render_mask(s["V"], s["tracer"])
        dV, = torch.autograd.grad(T.mask_loss(m, s["target"]), (s["V"],))
        return dict(mask=m.detach(), dV=dV)
    if kind == "step":
        leaves = {"V": s["V"], "ior": s["ior"]}
        if "mu" in s:
            leaves["mu"] = s["mu"]
            rgb = A.render_grid(s["V"], s["ior"], s["mu"], s["tracer"], s["lo"], s["hi"], s["samples"])
        elif "w" in s:
            leaves.update(sigma=s["sigma"], w=s["w"], b=s["b"])
            rgb = A.render_mlp(s["V"], s["ior"], s["sigma"], s["w"], s["b"], s["tracer"])
        else:
            leaves["sigma"] = s["sigma"]
            rgb = A.render(s["V"], s["ior"], s["sigma"], s["tracer"])
        grads = torch.autograd.grad(((rgb - s["target"]) ** 2).mean(), list(leaves.values()))
        return dict(zip(["rgb"] + ["d_" + k for k in leaves], [rgb.detach(), *grads]))
    if kind == "view":
        rgb, wtrunc, flags = B.dt_trace_forward(s["scene"], s["rays"], s["params"], s["buf"])
        return dict(rgb=rgb, wtrunc=wtrunc, flags=flags)
    s["mesh"].build()
    rgb, _, _ = B.dt_trace_forward(s["scene"], s["rays"], s["params"], s["buf"], want_aux=False)
    grad = (rgb - s["target"]) * (2.0 / rgb.numel())
    dV, d_ior, d_sigma = B.dt_trace_backward(s["scene"], s["rays"], s["params"], s["buf"], grad)
    out = dict(rgb=rgb, d_V=dV, d_ior=d_ior, d_sigma=d_sigma)
    if kind == "field":
        f = s["scene"].field
        out.update(d_grid=f.d_grid, d_planes=f.d_planes, d_texels=s["scene"].env.d_texels)
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: every input array read once, every output written once.
    Operations: per ray segment (about depth + 1 of them per camera ray on
    these scenes) the box tests of one path down the tree, one triangle test
    and the shading; three times that where gradients are asked for; the
    environment network's multiply-adds per camera ray; per sample of a grid
    or field its interpolation."""
    kind = case["kind"]
    if kind == "serve":
        rows = _serve_requests(case, 0)
        px = sum(r[2] ** 2 for r in rows)
        seg = sum(r[2] ** 2 * (r[3] + 1) for r in rows)
        nf = sum(2 * a * b for a, b in SERVE_FACES)
        return {"bytes": 24 * px + 30 * nf, "flops": seg * (20 * 17 + 200)}
    nv, nf = _faces(case)
    mesh = 12 * nv + 12 * nf
    if kind == "solve":
        # unknowns in, vertices out, the edge lists; the product with the
        # matrix once for each of about sqrt(condition) * 12 iterations
        its = 12 * math.sqrt(1 + 12 * case["lam"])
        return {"bytes": 24 * nv + 8 * 3 * nv, "flops": its * nv * 3 * (2 * 6 + 8)}
    if kind == "build":
        return {"bytes": mesh + 24 * nf + 12 * nv + 48 * case["picks"], "flops": nf * (40 + 12 * math.log2(nf))}
    rays = case["rays"] if kind == "batch" else case.get("views", 1) * case["width"] * case["height"]
    if kind == "mask":
        return {"bytes": mesh + 12 * nv + 8 * rays, "flops": rays * (20 * math.log2(nf) + 60) + 3 * nf * 30}
    seg = rays * (case["depth"] + 1)
    per = 20 * math.log2(nf) + 200
    nbytes, flops = mesh + 12 * rays + (24 * rays if kind == "batch" else 0), seg * per
    if kind != "view":
        nbytes, flops = nbytes + 12 * nv + 12 * rays, 3 * flops
    if case.get("env") == "mlp" or kind == "shell":
        layers, w = case.get("layers", 3), case.get("hidden", 64)
        flops += 3 * rays * 2 * (39 * w + (layers - 1) * w * w + 3 * w)
    else:
        nbytes += 12 * 512 * 256
    if case.get("grid"):
        taps = 20 * 8 if kind == "field" else 8 * 6
        flops += 3 * seg / 2 * case["samples"] * taps
        nbytes += 2 * 16 * case["grid"] ** 3
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
def _normals(V, F):
    """One third of the sum of the unit normals of the faces around each vertex."""
    p0, p1, p2 = V[F[:, 0]], V[F[:, 1]], V[F[:, 2]]
    n = torch.linalg.cross(p1 - p0, p2 - p0)
    n = n / n.norm(dim=-1, keepdim=True)
    acc = torch.zeros_like(V)
    for k in range(3):
        acc = acc.index_add(0, F[:, k], n)
    return acc / 3.0


@torch.no_grad()
def _closest(o, d, V, F, skip):
    """Nearest face along each ray (-1: none), every face tested."""
    p0, e1, e2 = V[F[:, 0]], V[F[:, 1]] - V[F[:, 0]], V[F[:, 2]] - V[F[:, 0]]
    N = torch.linalg.cross(e1, e2)
    m1, m2 = torch.linalg.cross(p0, e1), torch.linalg.cross(p0, e2)
    c0 = (p0 * N).sum(-1)
    tri = torch.full((len(o),), -1, dtype=torch.int64, device=o.device)
    step = max(1, 40_000_000 // len(F))
    for a in range(0, len(o), step):
        oo, dd = o[a:a + step], d[a:a + step]
        det = -(dd @ N.T)
        m = torch.linalg.cross(dd, oo)
        u = (dd @ m2.T - m @ e2.T) / det
        v = (m @ e1.T - dd @ m1.T) / det
        t = (oo @ N.T - c0) / det
        t[(u < 0) | (v < 0) | (u + v > 1) | ~(t > 1e-5)] = math.inf
        rows = torch.arange(len(oo), device=o.device)
        sk = skip[a:a + step]
        t[rows[sk >= 0], sk[sk >= 0]] = math.inf
        best, at = t.min(1)
        tri[a:a + step] = torch.where(torch.isfinite(best), at, -1)
    return tri


def _meet(o, d, V, F, tri):
    """Distance and barycentrics on the given faces, differentiable."""
    p0, p1, p2 = (V[F[tri, k]] for k in range(3))
    e1, e2, s = p1 - p0, p2 - p0, o - p0
    pv = torch.linalg.cross(d, e2)
    inv = 1.0 / (e1 * pv).sum(-1)
    qv = torch.linalg.cross(s, e1)
    return (e2 * qv).sum(-1) * inv, (s * pv).sum(-1) * inv, (d * qv).sum(-1) * inv


def _sky(tex, d):
    """Bilinear equirect lookup (row 0 at +y, wrapping in azimuth)."""
    H, W = tex.shape[:2]
    x = (torch.atan2(d[:, 0], -d[:, 2]) / (2 * math.pi) + 0.5) * W - 0.5
    y = torch.atan2(torch.sqrt(d[:, 0] ** 2 + d[:, 2] ** 2), d[:, 1]) / math.pi * H - 0.5
    x0, y0 = x.detach().floor(), y.detach().floor()
    fx, fy = (x - x0)[:, None], (y - y0)[:, None]
    xa, xb = (x0.long() % W), ((x0.long() + 1) % W)
    ya, yb = y0.long().clamp(0, H - 1), (y0.long() + 1).clamp(0, H - 1)
    return ((tex[ya, xa] * (1 - fx) + tex[ya, xb] * fx) * (1 - fy) + (tex[yb, xa] * (1 - fx) + tex[yb, xb] * fx) * fy)


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _render64(V, F, o, d, ior, sigma, tex, depth):
    """Pixel colours and truncated weights of the split-ray recursion, one ray a pixel."""
    n = len(o)
    rgb, wtrunc = torch.zeros_like(o), torch.zeros_like(o)
    vn = _normals(V, F)
    pix, w = torch.arange(n, device=o.device), torch.ones_like(o)
    skip = torch.full((n,), -1, dtype=torch.int64, device=o.device)
    for g in range(depth + 1):
        if not len(o):
            break
        tri = _closest(o.detach(), d.detach(), V.detach(), F, skip)
        miss, hit = tri < 0, tri >= 0
        rgb = rgb.index_add(0, pix[miss], w[miss] * _sky(tex, d[miss]))
        o, d, w, pix, tri = o[hit], d[hit], w[hit], pix[hit], tri[hit]
        t, b1, b2 = _meet(o, d, V, F, tri)
        x = o + d * t[:, None]
        p = [V[F[tri, k]] for k in range(3)]
        ng = torch.linalg.cross(p[1] - p[0], p[2] - p[0])
        enter = (d * ng).sum(-1) < 0
        sgn = torch.where(enter, 1.0, -1.0).to(V.dtype)[:, None]
        nrm = _unit(sum(vn[F[tri, k]] * b[:, None] for k, b in enumerate((1 - b1 - b2, b1, b2)))) * sgn
        away = (d * nrm).sum(-1) >= 0
        nrm = torch.where(away[:, None], _unit(ng) * sgn, nrm)
        ci = -(d * nrm).sum(-1)
        w = w * torch.where(enter[:, None], torch.ones_like(w), torch.exp(-sigma * t[:, None]))
        if g == depth:
            wtrunc = wtrunc.index_add(0, pix, w)
            break
        one = torch.ones_like(ci)
        ei, et = torch.where(enter, one, ior * one), torch.where(enter, ior * one, one)
        er = et / ei
        s2 = (1 - ci * ci) / (er * er)
        tir = s2 > 1
        ct = torch.sqrt(torch.where(tir, one, 1 - s2))
        rs, rp = (ei * ci - et * ct) / (ei * ci + et * ct), (ei * ct - et * ci) / (ei * ct + et * ci)
        R = torch.where(tir, one, 0.5 * (rs * rs + rp * rp))
        dr = _unit(d + nrm * (2 * ci)[:, None])
        go = ~tir
        dt = _unit((d / er[:, None] + nrm * (ci / er - ct)[:, None])[go])
        o, d = torch.cat([x, x[go]]), torch.cat([dr, dt])
        w = torch.cat([w * R[:, None], (w * (1 - R)[:, None])[go]])
        pix, skip = torch.cat([pix, pix[go]]), torch.cat([tri, tri[go]])
    return rgb, wtrunc


def _camera_rays64(c):
    """Rays through the pixel centres of a camera."""
    e, f = np.array(c.eye), np.array(c.target) - np.array(c.eye)
    f /= np.linalg.norm(f)
    r = np.cross(f, c.up)
    r /= np.linalg.norm(r)
    u = np.cross(r, f)
    th = math.tan(math.radians(c.fov_deg) / 2)
    px = (2 * (np.arange(c.width) + 0.5) / c.width - 1) * th * c.width / c.height
    py = (1 - 2 * (np.arange(c.height) + 0.5) / c.height) * th
    d = f + r * px[None, :, None] + u * py[:, None, None]
    d = (d / np.linalg.norm(d, axis=-1, keepdims=True)).reshape(-1, 3)
    return np.broadcast_to(e, d.shape).copy(), d


def _edges(F):
    e = torch.cat([F[:, [0, 1]], F[:, [1, 2]], F[:, [2, 0]]]).long()
    return torch.unique(torch.sort(e, 1).values, dim=0)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("serve", "step", "field", "shell", "mask"):
        return None   # millions of rays against every face: too long in 64 bits
    Vn, Fn = _mesh(case, seed)
    V, F = _dev(Vn).double(), _dev(Fn).long()
    if kind == "solve":
        e = _edges(F)
        i, j = torch.cat([e[:, 0], e[:, 1]]), torch.cat([e[:, 1], e[:, 0]])
        deg = torch.bincount(i, minlength=len(V)).double()[:, None]

        def mul(x):
            return x + case["lam"] * (deg * x - torch.zeros_like(x).index_add(0, i, x[j]))
        # the unknowns as the optimiser holds them: float32
        b = mul(V).float().double()
        x = torch.zeros_like(b)
        r = b.clone()
        p, rr = r.clone(), (r * r).sum(0)
        for _ in range(4000):
            q = mul(p)
            a = rr / (p * q).sum(0)
            x, r = x + a * p, r - a * q
            new = (r * r).sum(0)
            if bool((new <= 1e-26 * (b * b).sum(0)).all()):
                break
            p, rr = r + new / rr * p, new
        return x
    if kind == "build":
        if case["picks"] * len(F) > 2e10:
            return dict(normals=_normals(V, F), tri=None, t=None, b=None)
        o, d = (_dev(a).double() for a in _batch_rays(case["picks"], seed))
        tri = _closest(o, d, V, F, torch.full((len(o),), -1, dtype=torch.int64, device=DEV))
        t, b1, b2 = _meet(o, d, V, F, tri.clamp_min(0))
        miss = tri < 0
        return dict(normals=_normals(V, F), tri=None, t=torch.where(miss, math.inf, t),
                    b=torch.where(miss[:, None], 0.0, torch.stack([b1, b2], -1)))
    n = case["rays"] if kind == "batch" else case["width"] * case["height"]
    if n * (case["depth"] + 2) * 1.5 * len(F) > 2e10:
        return None
    ior, sigma = (x.double() for x in _material(seed))
    small = kind == "view" and case["mesh"] == "icosphere"
    tex = _dev(synth.env_equirect(64 if small else 512, 32 if small else 256, seed=seed)).double()
    if kind == "view":
        o, d = (_dev(a) for a in _camera_rays64(_cameras(case, seed)[0]))
        rgb, wtrunc = _render64(V, F, o, d, ior, sigma, tex, case["depth"])
        return dict(rgb=rgb, wtrunc=wtrunc, flags=None)
    o, d = (_dev(a).double() for a in _batch_rays(n, seed))
    d = d.clone()
    leaves = [x.requires_grad_(True) for x in (V, ior, sigma)]
    rgb, _ = _render64(V, F, o, d, ior, sigma, tex, case["depth"])
    target = _target(n, seed).double()
    dV, d_ior, d_sigma = torch.autograd.grad(((rgb - target) ** 2).mean(), leaves)
    return dict(rgb=rgb.detach(), d_V=dV, d_ior=d_ior, d_sigma=d_sigma)
