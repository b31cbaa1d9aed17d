"""The pixels that the bipyramids of the vertex-gradient test leave out (a shading
normal on the wrong side, or a ray that leaves the object from inside) are those
that the oracle itself leaves undefined, under a third, and no others."""
import numpy as np
import pytest

from paper_2603_00413_amd import synth
from tests.gpu_helpers import UNDEFINED, Pair, check_radiance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sides", [3, 8, 9, 40])
def test_defined_share(sides):
    a = 2 * np.pi * np.arange(sides) / sides
    V = np.concatenate([np.stack([np.cos(a), np.sin(a), 0.05 * np.sin(3 * a)], 1),
                        [[0.02, 0.01, 0.9], [0.01, -0.03, -0.8], [0.3, 0.3, 5.0]]])
    k = np.arange(sides)
    n = (k + 1) % sides
    F = np.concatenate([np.stack([k, n, 0 * k + sides], 1), np.stack([n, k, 0 * k + sides + 1], 1)]).astype(np.int32)
    cams = [synth.look_at_camera(e, 40, 40) for e in synth.views_on_sphere(2, 3.0, seed=5)]
    P = Pair(V, F, 1.4, 0.3, synth.env_equirect(128, 64, seed=2), cams, 3)
    _, rgb, _, fl = P.gpu_forward(tape=False)
    own = ((P.orc.trace(P.o, P.d)["flags"] & UNDEFINED) != 0).mean()
    assert own < 1 / 3
    check_radiance(P.orc, P.o, P.d, rgb, fl, P.sig, label=f"bipyramid {sides}", max_excluded=own + 1 / len(fl))
