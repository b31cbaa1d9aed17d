"""The tree build at the sizes where its kernels change: tiles of 512 sorted
triangles (one tile, one more, several that climb through shared nodes), the
short radix sort (1,024 to 131,072 faces) and its general form, the one-block
scan.  The tree must give brute force's hits, and the vertex normals those of a
plain float64 sum."""
import numpy as np
import pytest
import torch

from paper_2603_00413_amd import binding as B
from paper_2603_00413_amd import synth
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


def _mesh(nf, seed):
    """nf faces of a displaced torus, a random subset in random order"""
    nu = max(8, int(np.ceil(np.sqrt(nf))) + 1)
    V, F = synth.displaced_torus(seed=seed, nu=nu, nv=(nf + 2 * nu - 1) // (2 * nu) + 3)
    F = F[np.random.default_rng(seed).permutation(len(F))[:nf]]
    return V.astype(np.float32), np.ascontiguousarray(F)


@pytest.mark.parametrize("nf", [511, 512, 513, 1023, 1024, 1025, 4097, 131072, 131073, 263000])
def test_build_sizes(nf):
    dev = device()
    V, F = _mesh(nf, nf % 97)
    assert len(F) == nf
    m = B.Mesh(torch.from_numpy(V).to(dev), torch.from_numpy(F).to(dev))
    P = V.astype(np.float64)
    n = np.cross(P[F[:, 1]] - P[F[:, 0]], P[F[:, 2]] - P[F[:, 0]])
    n /= np.linalg.norm(n, axis=1, keepdims=True)
    N = np.zeros_like(P)
    for k in range(3):
        np.add.at(N, F[:, k], n)
    # float32 face normals (a few ulps each, up to cancellation in the cross
    # product of edges much shorter than the coordinates), summed over a ring
    assert np.abs(m.vertex_normals().cpu().numpy() - N / 3).max() <= 1e-3
    rng = np.random.default_rng(nf)
    k = 2048 if nf > 5000 else 6000
    o = rng.normal(size=(k, 3)).astype(np.float32) * 2.0
    c = V[F[rng.integers(0, nf, k)]].mean(1)
    d = (c + rng.normal(0.0, 0.01, (k, 3)) - o).astype(np.float32)
    sc = B.Scene(m, torch.ones(1, device=dev), torch.zeros(3, device=dev), B.Env(torch.ones(4, 8, 3, device=dev)))
    args = [torch.from_numpy(x).to(dev) for x in (o, d)]
    got = [x.cpu().numpy() for x in B.dt_intersect(sc, *args)]
    ref = [x.cpu().numpy() for x in B.dt_intersect(sc, *args, brute_force=True)]
    assert (ref[0] >= 0).mean() > 0.3
    assert np.array_equal(got[0], ref[0])
    hit = ref[0] >= 0
    assert np.array_equal(got[1][hit], ref[1][hit]) and np.array_equal(got[2][hit], ref[2][hit])
    # the same mesh again gives the same tree
    blob = m.blob.clone()
    m.build()
    assert torch.equal(blob, m.blob)
