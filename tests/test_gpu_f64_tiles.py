"""FP64 chi sum at the edges of its 32 and 64 wide tiles and of its 8-pair
stages, against the oracle; values that are not finite mark their row and column
only.

Bound.  A sum of 2 K real products w a b, in any order, is off by at most
(2 K + 2) 2^-53 sum |w a b|; the oracle's is too, and Re and Im have such a sum each.
"""

import numpy as np
import pytest

import oracle
from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def run(torch, M, ev, ec, omega):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    (chi,) = h.chi0([dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=ev.shape[0], nv=ev.shape[1], nc=ec.shape[1], head=-1,
                          prefactor=0.5)], omega)
    torch.cuda.synchronize()
    out = chi.cpu().numpy()
    h.close()
    return out


@pytest.mark.parametrize("nk,nv,nc,ng", [(1, 1, 1, 1), (1, 1, 7, 31), (1, 1, 8, 32), (1, 3, 3, 33), (1, 2, 20, 63),
                                         (3, 5, 11, 65), (2, 31, 33, 97), (5, 17, 29, 191), (1, 40, 64, 577),
                                         (1, 3, 5, 1281)])
def test_edges(torch_dev, nk, nv, nc, ng):
    rng = np.random.default_rng(nc + ng)
    K = nk * nv * nc
    M = rng.standard_normal((K, ng)) + 1j * rng.standard_normal((K, ng))
    ev, ec = np.sort(rng.uniform(-10, 0, (nk, nv))), np.sort(rng.uniform(1, 20, (nk, nc)))
    om = np.array([0.0, 3.0])
    w = oracle.weights(ev, ec, om)
    ref = oracle.chi(M, w, 0.5)
    got = run(torch_dev, M, ev, ec, om)
    size = np.abs(M.real) + np.abs(M.imag)
    for i in range(len(om)):
        mass = 0.5 * (size * np.abs(w[i]).reshape(K, 1)).T @ size
        assert np.all(np.abs(got[i] - ref[i]) <= 2 * (2 * K + 8) * 2.0 ** -53 * mass)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("K,ng,at", [(1, 33, (0, 32)), (13, 70, (12, 64)), (800, 130, (517, 40))])
def test_not_finite(torch_dev, value, K, ng, at):
    rng = np.random.default_rng(3)
    M = rng.standard_normal((K, ng)) + 1j * rng.standard_normal((K, ng))
    M[at] = 1.0 + 1j * value
    got = run(torch_dev, M, np.array([[-1.0]]), np.sort(rng.uniform(1, 20, (1, K))), [0.0])[0]
    bad = np.zeros((ng, ng), dtype=bool)
    bad[at[1], :] = bad[:, at[1]] = True
    assert np.array_equal(~np.isfinite(got.real), bad)
