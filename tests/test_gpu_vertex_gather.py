"""Vertex gradients where a vertex has fewer or more faces than the lanes that
gather them: bipyramids with apexes of 3, 8, 9 and 40 faces, and a vertex of no
face at all.  Against the oracle, element by element, on the pixels whose paths
it defines (vertex normals this far from the faces leave a good part undefined)."""
import numpy as np
import pytest

from paper_2603_00413_amd import synth
from tests.gpu_helpers import GradRef, Pair, check_elements, check_material, check_radiance, gradient_pixels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sides", [3, 8, 9, 40])
def test_bipyramid(sides):
    a = 2 * np.pi * np.arange(sides) / sides
    V = np.concatenate([np.stack([np.cos(a), np.sin(a), 0.05 * np.sin(3 * a)], 1),
                        [[0.02, 0.01, 0.9], [0.01, -0.03, -0.8], [0.3, 0.3, 5.0]]])
    k = np.arange(sides)
    n = (k + 1) % sides
    F = np.concatenate([np.stack([k, n, 0 * k + sides], 1), np.stack([n, k, 0 * k + sides + 1], 1)]).astype(np.int32)
    cams = [synth.look_at_camera(e, 40, 40) for e in synth.views_on_sphere(2, 3.0, seed=5)]
    P = Pair(V, F, 1.4, 0.3, synth.env_equirect(128, 64, seed=2), cams, 3)
    buf, rgb, _, fl = P.gpu_forward(tape=True)
    chk = check_radiance(P.orc, P.o, P.d, rgb, fl, P.sig, label=f"bipyramid {sides}", max_excluded=1.0)
    gr = GradRef(P.orc, P.o, P.d, chk["ref"]["sig"])
    g = np.random.default_rng(sides).normal(size=rgb.shape) * gradient_pixels(chk, fl, gr.stable)[:, None]
    dV, de, ds = P.gpu_backward(buf, g)
    o, oa, sp = gr.grads(g)
    check_elements(dV, o["dV"], oa["dV"], f"bipyramid {sides} dV", sp["dV"])
    check_material(de, ds, o, oa, sp, f"bipyramid {sides}")
    assert (dV[-1] == 0).all()
