"""Images are copied out beside the steps that follow: with a pixel pool that
every next request needs as soon as it is released, each image is still the one
its request rendered (path signatures exactly, radiance to the order of a
pixel's sum), as a server with room for all gives it."""
import numpy as np
import pytest

from paper_2603_00413_amd import synth
from paper_2603_00413_amd.serve import Request, Server
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res,images", [(256, 1), (200, 2)])
def test_pool_reused_under_copies(res, images):
    device()
    V, F = synth.displaced_torus(seed=5, nu=60, nv=30)
    eyes = synth.views_on_sphere(8, 3.0, seed=3)

    def serve(pool):
        srv = Server(queue_capacity=1 << 20, pixel_pool=pool)
        srv.add_scene(V, F, 1.45, 0.3, synth.env_equirect(64, 32, seed=2))
        return srv.run([Request(k, 0, synth.look_at_camera(e, res, res), 4, None, arrival=0.0)
                        for k, e in enumerate(eyes)], realtime=False)

    for a, b in zip(serve(images * res * res), serve(len(eyes) * res * res)):
        assert (a.sig == b.sig).all()
        # a pixel sums at most 2^4 paths, in any order
        assert np.abs(a.image - b.image).max() <= 2**4 * 2**-23 * np.abs(b.image).max()
