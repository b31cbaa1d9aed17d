"""The field's backward where its sums can go wrong: a field of one cell (every
record of a wave in one sum), one of mostly distinct cells, one sample per
segment, generations of fewer nodes than a wave holds, and rays' gradients with
the field itself held fixed.  Against the FP64 oracle, element by element, at
the oracle's FP32 rounding bounds."""
import numpy as np
import pytest

from paper_2603_00413_amd import binding as B
from tests.gpu_helpers import DV_ORDER_TOL, icosphere_pair
from tests.test_gpu_field import HI, HI_WIDE, LO, LO_WIDE, _grad_check, _with_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,res,samples,box,px", [
    ((2, 2, 2), 2, 8, (LO, HI), 64),                # one grid cell, one cell per plane
    ((2, 3, 9), 3, 1, (LO_WIDE, HI_WIDE), 64),      # one sample; rays start inside the box
    ((33, 31, 29), 41, 7, (LO, HI), 64),            # nearly every record a cell of its own
    ((5, 6, 4), 7, 5, (LO, HI), 9),                 # 81 camera rays: a full wave and a short one
    ((5, 6, 4), 7, 5, (LO, HI), 5),                 # 25: less than a wave
])
def test_field_sums(n, res, samples, box, px):
    P = _with_field(icosphere_pair(sigma=(0.5, 0.2, 0.1), res=px), seed=21, samples=samples, n=n, res=res, box=box)
    _grad_check(P, seed=22, label=f"field {n} planes {res} S={samples} {px}x{px}")


def test_fixed_field_gives_the_same_vertex_gradient():
    """Without d_grid / d_planes the adjoint takes the same ray terms."""
    P = _with_field(icosphere_pair(sigma=(0.5, 0.2, 0.1)), seed=23, samples=6)
    buf, rgb, _, _ = P.gpu_forward(tape=True)
    g = np.random.default_rng(24).normal(size=rgb.shape)
    dV1, de1, ds1 = P.gpu_backward(buf, g)
    f = P.field
    P.field = B.Field(f.grid, f.planes, f.lo, f.hi, f.samples, want_grad=False)
    P.scene = B.Scene(P.mesh, P.ior_t, P.sigma_t, P.env, field=P.field)
    buf, _, _, _ = P.gpu_forward(tape=True)
    dV2, de2, ds2 = P.gpu_backward(buf, g)
    assert np.linalg.norm(dV1 - dV2) <= DV_ORDER_TOL * np.linalg.norm(dV1)
    assert abs(de1 - de2) <= 1e-6 * abs(de1) + 1e-9
