"""The environment MLP's kernels at the sizes where they can go wrong: fewer
directions than a wave or a block takes, every width and depth, the smallest and
largest encodings, weights that start at an odd address, and the weight gradient
of short miss lists.  Against the oracle's FP64 network at the bars that its
value and gradients are held to elsewhere."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import GradRef, Pair, check_elements, check_radiance, device, gradient_pixels, rgb_rel_err

pytestmark = pytest.mark.gpu


def _net(seed, layers, width, n_freq):
    Ws, Bs = synth.env_mlp_weights(seed=seed, n_layers=layers, width=width, n_freq=n_freq)
    oenv = oracle.Env(mlp=([w.astype(np.float64) for w in Ws], [b.astype(np.float64) for b in Bs], n_freq))
    return Ws, Bs, oenv


@pytest.mark.parametrize("width,layers,n_freq,n", [
    (64, 1, 0, 1), (64, 2, 7, 15), (64, 3, 6, 17), (64, 4, 3, 129), (128, 1, 7, 16), (128, 2, 0, 33), (128, 3, 6, 127),
    (128, 4, 6, 1000)])
def test_query_shapes(width, layers, n_freq, n):
    dev = device()
    Ws, Bs, oenv = _net(11 * layers + width, layers, width, n_freq)
    env = B.Env.mlp(Ws, Bs, n_freq, dev)
    rng = np.random.default_rng(n)
    d = rng.normal(size=(n, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    g = rng.normal(size=(n, 3)).astype(np.float32)
    dt, gt = torch.from_numpy(d).to(dev), torch.from_numpy(g).to(dev)
    E, gd = B.dt_env_query(env, dt), B.dt_env_query_backward(env, dt, gt)
    assert rgb_rel_err(E.cpu().numpy().astype(np.float64), oenv.eval(d.astype(np.float64))).max() <= 1e-4
    far = oenv.kink_margin(d.astype(np.float64)) > 1e-5
    gdo = oenv.eval_grad(d.astype(np.float64), g.astype(np.float64))
    r = np.linalg.norm(gd.cpu().numpy() - gdo, axis=1) / np.linalg.norm(gdo, axis=1)
    assert r[far].max(initial=0.0) <= 1e-3
    # the same weights two bytes further: the eight-at-a-time copy does not apply
    moved = torch.empty(env.weights.numel() + 8, dtype=torch.int16, device=dev)[1:1 + env.weights.numel()]
    moved.copy_(env.weights)
    assert moved.data_ptr() % 16 == 2
    env.s.weights = moved.data_ptr()
    assert torch.equal(B.dt_env_query(env, dt), E)
    assert torch.equal(B.dt_env_query_backward(env, dt, gt), gd)


@pytest.mark.parametrize("layers,px", [(2, 3), (3, 5), (4, 9)])
def test_weight_gradient_of_few_misses(layers, px):
    dev = device()
    wl = synth.icosphere_scene(sigma=(0.5, 0.2, 0.1), res=px)
    Ws, Bs, oenv = _net(5 + layers, layers, 64, 6)
    P = Pair(wl.V, wl.F, wl.ior, wl.sigma, wl.env, wl.cameras, wl.max_depth)
    P.env = B.Env.mlp(Ws, Bs, 6, dev, want_grad=True)
    P.scene = B.Scene(P.mesh, P.ior_t, P.sigma_t, P.env)
    P.orc = oracle.Scene(P.V32.astype(np.float64), P.F, float(P.ior), P.sigma.astype(np.float64), oenv, wl.max_depth)
    buf, rgb, _, fl = P.gpu_forward(tape=True)
    chk = check_radiance(P.orc, P.o, P.d, rgb, fl, P.sig, mlp=True, label=f"{layers} x 64 MLP, {px}^2")
    gr = GradRef(P.orc, P.o, P.d, chk["ref"]["sig"])
    g = np.random.default_rng(layers).normal(size=rgb.shape) * gradient_pixels(chk, fl, gr.stable)[:, None]
    P.gpu_backward(buf, g)
    dW, dB = P.env.split_grad()
    o, oa, sp = gr.grads(g, want_mlp=True)
    for l in range(layers + 1):
        check_elements(dW[l], o["d_mlp"][0][l], oa["d_mlp"][0][l], f"dW[{l}]", sp["d_mlp"][0][l], floor_frac=0.1)
        check_elements(dB[l], o["d_mlp"][1][l], oa["d_mlp"][1][l], f"db[{l}]", sp["d_mlp"][1][l], floor_frac=0.1)
