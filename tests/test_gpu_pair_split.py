"""Pair densities where the transform passes cut their x-planes and valence bands
finer than for a full chip, for every box of the lane-per-line passes and the 48^3
box of the mixed ones, with wavefunction spheres larger and smaller than the
dielectric one.

Bound.  M is a sum over the grid of conj(u_v) u_c, so an error in either factor
enters with the norm of the other: three transforms of at most 5 log2(48^3) 2^-53
each and sums of 48 terms, 512 2^-53 |c_v| |c_c| in all.
"""

import numpy as np
import pytest

import oracle
from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


def sphere(r2):
    r = int(np.sqrt(r2))
    a = np.arange(-r, r + 1)
    g = np.stack(np.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    return np.ascontiguousarray(g[(g ** 2).sum(1) <= r2].astype(np.int32))


@pytest.mark.parametrize("nk,nv,nc", [(1, 1, 1), (1, 5, 3), (3, 2, 17), (1, 13, 19)])
@pytest.mark.parametrize("n,rw2,re2", [(16, 18, 18), (24, 50, 37), (32, 82, 101), (48, 131, 131), (48, 145, 40)])
def test_split(n, rw2, re2, nk, nv, nc):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(n + nv)
    gw, ge = sphere(rw2), sphere(re2)
    rng.shuffle(ge)
    rnd = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    cv, cc = rnd(nk, nv, len(gw)), rnd(nk, nc, len(gw))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    M = h.pair_density((n, n, n), gw, ge, dev(cv), dev(cc))
    torch.cuda.synchronize()
    h.close()
    some = np.sort(rng.permutation(nk * nv * nc)[:5])
    ref = oracle.pair_density(gw, ge, cv, cc, pairs=some)
    size = np.einsum("kv,kc->kvc", np.linalg.norm(cv, axis=2), np.linalg.norm(cc, axis=2)).reshape(-1, 1)
    assert np.all(np.abs(M.cpu().numpy()[some] - ref) <= 512 * 2.0 ** -53 * size[some])
