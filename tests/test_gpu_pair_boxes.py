"""Every pair of pair-density calls on each box of the lane-per-line passes and on the
48^3 one of the mixed passes, valence bands in several blocks with a remainder; on 48^3
with the scratch of the band lines smaller and larger than the pairs' (max(nv, nc)
(2 rw + 1)^2 against nv nc (2 re + 1)^2), which decides the bands' path.

Bound.  M is a sum over the grid of conj(u_v) u_c, so an error in either factor enters
with the norm of the other: three transforms of at most 5 log2(48^3) 2^-53 each and
sums of 48 terms, 512 2^-53 |c_v| |c_c| in all.
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


CASES = [(16, 18, 18, 1, 13, 19), (24, 50, 37, 1, 13, 19), (32, 82, 101, 1, 13, 19), (24, 50, 37, 3, 7, 5),
         # |m| <= 14 and 7: 36 points and so the 48^3 box
         (48, 200, 60, 1, 1, 1), (48, 200, 60, 2, 3, 9), (48, 200, 60, 1, 4, 11), (48, 200, 60, 1, 13, 19),
         (48, 200, 60, 3, 5, 17)]


@pytest.mark.parametrize("n,rw2,re2,nk,nv,nc", CASES)
def test_every_pair(n, rw2, re2, nk, nv, nc):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(n + nv)
    gw, ge = sphere(rw2), sphere(re2)
    rng.shuffle(ge)
    assert list(bgw.pair_transform_box((n, n, n), gw, ge)) == [n, n, n]
    rnd = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    cv, cc = rnd(nk, nv, len(gw)), rnd(nk, nc, len(gw))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    M = h.pair_density((n, n, n), gw, ge, dev(cv), dev(cc))
    torch.cuda.synchronize()
    h.close()
    ref = oracle.pair_density(gw, ge, cv, cc)
    size = np.einsum("kv,kc->kvc", np.linalg.norm(cv, axis=2), np.linalg.norm(cc, axis=2)).reshape(-1, 1)
    assert np.all(np.abs(M.cpu().numpy() - ref) <= 512 * 2.0 ** -53 * size)
