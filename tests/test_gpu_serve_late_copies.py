"""Images whose copies are certainly still to come when their pixels are given
to the next request: the copy stream is held up by device copies of its own
before the run, so the first image's copy waits behind them while the server
admits on.  Each image and its flags are still the request's own."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import synth
from paper_2603_00413_amd.serve import Request, Server
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images", [1, 2])
def test_pixels_wait_for_the_copy(images, monkeypatch):
    dev = device()
    res = 128
    V, F = synth.displaced_torus(seed=5, nu=60, nv=30)
    eyes = synth.views_on_sphere(8, 3.0, seed=3)
    late = []
    wait = torch.cuda.Stream.wait_event

    def counted(stream, event):
        late.append(not event.query())
        return wait(stream, event)

    def serve(pool, held):
        srv = Server(queue_capacity=1 << 20, pixel_pool=pool)
        srv.add_scene(V, F, 1.45, 0.3, synth.env_equirect(64, 32, seed=2))
        reqs = [Request(k, 0, synth.look_at_camera(e, res, res), 4, None, arrival=0.0) for k, e in enumerate(eyes)]
        a, b = (torch.zeros(1 << 28, device=dev) for _ in range(2))
        torch.cuda.synchronize()
        if held:
            # some 0.4 ms each; a step takes a few tenths of one
            with torch.cuda.stream(srv._copies):
                for _ in range(100):
                    b.copy_(a)
        out = srv.run(reqs, realtime=False)
        torch.cuda.synchronize()
        return out

    want = serve(len(eyes) * res * res, False)
    monkeypatch.setattr(torch.cuda.Stream, "wait_event", counted)
    got = serve(images * res * res, True)
    assert any(late), "no admission met a copy still to come"
    for a, b in zip(got, want):
        assert (a.sig == b.sig).all() and (a.flags == b.flags).all()
        # a pixel sums at most 2^4 paths, in any order
        assert np.abs(a.image - b.image).max() <= 2**4 * 2**-23 * np.abs(b.image).max()
