"""Split-precision chi sum of columns whose magnitudes change along the pairs: a
value keeps its digits below the largest of its own run of 96 pairs, whatever the
neighbouring runs hold, in chi0 on both axes and in the exchange kernel.

Bound.  In a run a value is N = rint(x 2^(39-e)), with 2^e at most 2.01 2^3 times the
run's largest magnitude on the weighted side and 2.01 2 times on the other.  Rounding
both factors of a real product costs at most 2^-40 (2.01 8 + 2.01 2) maxA maxB, the
digit products left out 4.05 2^-40 (2.01 8) (2.01 2) maxA maxB: 283 2^-40 in all, over
the run's products; Re and Im are two real products each.
"""

import numpy as np
import pytest

import oracle
from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu

RUN = 96


@pytest.fixture(scope="module")
def torch_dev():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def by_run(x):
    """Largest magnitude of each run of pairs, [runs][columns]."""
    return np.stack([np.abs(x[t:t + RUN]).max(0) for t in range(0, len(x), RUN)])


def bound(M, w, pf):
    """Of one real weight vector: sum over runs of (pairs) 2 sqrt 2 283 2^-40 maxA maxB."""
    size = np.maximum(np.abs(M.real), np.abs(M.imag))
    a, b = by_run(np.abs(w)[:, None] * size), by_run(size)
    digits = pf * RUN * 2 * np.sqrt(2.0) * 283 * 2.0 ** -40 * (a.T @ b)
    # the oracle's and the sums' own FP64 rounding
    return digits + 1e-13 * pf * (np.abs(w)[:, None] * size * 2).T @ size


def columns(rng, K, ng, spread):
    """Columns whose magnitude jumps by up to 2^spread from one stretch of pairs to the next."""
    M = rng.standard_normal((K, ng)) + 1j * rng.standard_normal((K, ng))
    M *= np.exp2(rng.uniform(-spread, 0.0, (K // 31 + 1, ng)).repeat(31, 0)[:K])
    M[: K // 2, 1] *= 2.0 ** -spread
    M[K // 2:, 2] *= 2.0 ** -spread
    M[RUN:2 * RUN, 3] = 0.0
    M[:, 4] = 0.0
    return M


@pytest.mark.parametrize("axis", ["imag", "advanced"])
@pytest.mark.parametrize("nk,nv,nc,ng", [(1, 1, 384, 5), (1, 1, 385, 97), (1, 2, 97, 64), (3, 5, 101, 193), (4, 7, 53, 130)])
@pytest.mark.parametrize("spread", [2.0, 5.0, 20.0, 60.0])
@pytest.mark.parametrize("slice_bytes", [None, "1"])  # "1": one launch per least range of pairs, later ones adding
def test_columns(torch_dev, nk, nv, nc, ng, spread, axis, slice_bytes, monkeypatch):
    if slice_bytes:
        monkeypatch.setenv("BGW_SPLIT_SLICE_BYTES", slice_bytes)
    rng = np.random.default_rng(nc + ng)
    K = nk * nv * nc
    M = columns(rng, K, ng, spread)
    # c fastest, energies over two decades: the weights change along the pairs too
    ev, ec = np.sort(rng.uniform(-1, 0, (nk, nv))), np.sort(np.exp(rng.uniform(0.0, 5.0, (nk, nc))))
    om = np.array([0.0, 3.0])
    if axis == "imag":
        w = oracle.weights(ev, ec, om)
        parts = [[x] for x in w]
    else:
        w = oracle.weights_real(ev, ec, om, 0.3, axis)
        parts = [[x.real, x.imag] for x in w]
    ref = oracle.chi(M, w, 0.5)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    (chi,) = h.chi0([dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=nk, nv=nv, nc=nc, head=-1, prefactor=0.5)], om,
                    precision=bgw.SPLIT_BF16, axis=axis, broadening=0.3)
    torch_dev.cuda.synchronize()
    got = chi.cpu().numpy()
    h.close()
    for i in range(len(om)):
        up = np.triu(sum(bound(M, x, 0.5) for x in parts[i]))  # the weighted side is the upper triangle's row
        up = up + np.triu(up, 1).T
        assert np.all(np.abs(got[i] - ref[i]) <= up)


@pytest.mark.parametrize("ratio", [1.0, 1e2, 1e4, 1e6])
def test_large_at_different_pairs(torch_dev, ratio):
    """One column large in the first 96 of 384 pairs, another in the last 96: their element
    of chi is as accurate, against its own products, as for columns alike in every pair."""
    rng = np.random.default_rng(int(ratio))
    K, ng = 384, 2
    M = rng.uniform(0.5, 1.0, (K, ng)) + 0j  # one sign: the sum is the sum of magnitudes
    M[96:, 0] /= ratio
    M[:288, 1] /= ratio
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    ev, ec = np.array([[-1.0]]), np.full((1, K), 3.0)
    h = bgw.Handle(0)
    (chi,) = h.chi0([dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=1, nv=1, nc=K, head=-1, prefactor=1.0)], [0.0],
                    precision=bgw.SPLIT_BF16)
    torch_dev.cuda.synchronize()
    got = chi.cpu().numpy()[0]
    h.close()
    ref = oracle.chi(M, oracle.weights(ev, ec, np.array([0.0])), 1.0)[0]
    # values of a run differ by a factor of 2 at most, so that its largest product is at most 4 of any
    assert abs(got[0, 1] - ref[0, 1]) <= 283 * 2.0 ** -40 * 4 * abs(ref[0, 1])


@pytest.mark.parametrize("spread", [3.0, 20.0])
def test_exchange_kernel(torch_dev, spread):
    """Kx contracts over G, where v falls from a large G = 0 term on."""
    rng = np.random.default_rng(int(spread))
    K, ng = 150, 611
    M = columns(rng, ng, K, spread).T.copy()  # [pairs][G], magnitudes changing along G
    v = np.exp2(-np.arange(ng) / 40.0)
    v[0] = 1e6
    h = bgw.Handle(0)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    kx = h.bse_kx(dev(M), dev(v), head=-1, prefactor=0.5, precision=bgw.SPLIT_BF16)
    torch_dev.cuda.synchronize()
    got = kx.cpu().numpy()
    h.close()
    ref = oracle.bse_kx(M, v, -1, 0.5)
    up = np.triu(bound(M.T.copy(), v, 0.5))
    up = up + np.triu(up, 1).T
    assert np.all(np.abs(got - ref) <= up)


def test_advanced_is_the_adjoint(torch_dev):
    """Weights, digits and INT32 sums are the same on both real axes: chi^a is chi^r's
    adjoint to the last bit."""
    rng = np.random.default_rng(4)
    nk, nv, nc, ng = 2, 3, 83, 130
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    q = dict(M=dev(columns(rng, nk * nv * nc, ng, 8.0)), ev=dev(np.sort(rng.uniform(-5, 0, (nk, nv)))),
             ec=dev(np.sort(rng.uniform(0.5, 9, (nk, nc)))), nk=nk, nv=nv, nc=nc, head=0, prefactor=0.5)
    h = bgw.Handle(0)
    r, a = (h.chi0([q], [0.0, 2.0, 7.0], precision=bgw.SPLIT_BF16, axis=x, broadening=0.2)[0]
            for x in ("retarded", "advanced"))
    torch_dev.cuda.synchronize()
    h.close()
    assert torch_dev.equal(a, r.mH.contiguous())


@pytest.mark.parametrize("nw", [3, 4, 5, 9])
def test_vectors_of_a_round(torch_dev, nw):
    """Exponents of the weighted side are found four vectors a round: counts around
    that, on weights of different ranges, and one that is not finite spoils its own
    vector only."""
    rng = np.random.default_rng(nw)
    K, ng = 450, 70
    M = columns(rng, K, ng, 6.0)
    ev, ec = np.array([[-0.5]]), np.sort(np.exp(rng.uniform(0.0, 5.0, (1, K))))
    om = np.concatenate([[0.0], np.exp2(rng.uniform(-3.0, 7.0, nw - 1))])
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    q = dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=1, nv=1, nc=K, head=-1, prefactor=0.5)
    (chi,) = h.chi0([q], om, precision=bgw.SPLIT_BF16)
    w = oracle.weights(ev, ec, om)
    ref = oracle.chi(M, w, 0.5)
    got = chi.cpu().numpy()
    for i in range(nw):
        up = np.triu(bound(M, w[i], 0.5))
        up = up + np.triu(up, 1).T
        assert np.all(np.abs(got[i] - ref[i]) <= up)
    ec[0, 200] = ev[0, 0]  # Delta = 0: the static weight is infinite, the others are zero
    (chi,) = h.chi0([dict(q, ec=dev(ec))], om, precision=bgw.SPLIT_BF16)
    torch_dev.cuda.synchronize()
    got = chi.cpu().numpy()
    h.close()
    assert not np.isfinite(got[0].real).any()
    assert np.isfinite(got[1:]).all()
