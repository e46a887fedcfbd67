"""Split-precision chi sum at the edges of its tiles, k-steps (32 pairs) and
digit chunks (384 pairs), against the oracle, within the bound of its digit
arithmetic; values that are not finite mark their row and column only.

Bound.  A value is N = rint(x 2^(39-e)), with 2^e at most 2.01 times the largest
magnitude of its chunk column: rounding both factors of a real product costs at
most 2^39 units of 2^(eA+eB-78), the digit products left out at most 2^40, so
3 2^-39 2.01^2 maxA maxB in all; Re and Im are two real products each.
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


def run(torch, M, ev, ec, omega, axis="imag", head=-1, precision=bgw.SPLIT_BF16):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = bgw.Handle(0)
    (chi,) = h.chi0([dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=ev.shape[0], nv=ev.shape[1], nc=ec.shape[1], head=head,
                          prefactor=0.5)], omega, precision=precision, axis=axis, broadening=0.3)
    torch.cuda.synchronize()
    out = chi.cpu().numpy()
    h.close()
    return out


@pytest.mark.parametrize("axis", ["imag", "advanced"])
@pytest.mark.parametrize("nk,nv,nc,ng", [(1, 1, 1, 1), (1, 1, 31, 63), (1, 3, 11, 65), (1, 2, 48, 96), (1, 1, 383, 97),
                                         (5, 7, 11, 128), (5, 7, 23, 193), (2, 20, 40, 191)])
@pytest.mark.parametrize("slice_bytes", [None, "1"])  # "1": one launch per least chunk range, later ones adding
def test_edges(torch_dev, nk, nv, nc, ng, axis, slice_bytes, monkeypatch):
    if slice_bytes:
        monkeypatch.setenv("BGW_SPLIT_SLICE_BYTES", slice_bytes)
    rng = np.random.default_rng(nc + ng)
    K = nk * nv * nc
    M = rng.standard_normal((K, ng)) + 1j * rng.standard_normal((K, ng))
    M *= np.exp(rng.uniform(-6.0, 6.0, (1, ng)))
    ev, ec = np.sort(rng.uniform(-10, 0, (nk, nv))), np.sort(rng.uniform(1, 20, (nk, nc)))
    om = np.array([0.0, 3.0])
    if axis == "imag":
        w = oracle.weights(ev, ec, om)
        parts = np.abs(w)
    else:
        w = oracle.weights_real(ev, ec, om, 0.3, axis)
        parts = np.abs(w.real) + np.abs(w.imag)
    ref = oracle.chi(M, w, 0.5)
    got = run(torch_dev, M, ev, ec, om, axis)
    for i in range(len(om)):
        wmax = float(parts[i].max())
        mx = np.maximum(np.abs(M.real), np.abs(M.imag)).max(0)
        bound = 0.5 * K * 2 * np.sqrt(2.0) * 3 * 2.0 ** -39 * 2.01 ** 2 * wmax * np.outer(mx, mx)
        # the oracle's and the sums' own FP64 rounding
        bound += 1e-13 * 0.5 * K * wmax * 2 * np.outer(mx, mx)
        assert np.all(np.abs(got[i] - ref[i]) <= bound)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_not_finite(torch_dev, value):
    rng = np.random.default_rng(3)
    K, ng = 800, 130
    M = rng.standard_normal((K, ng)) + 1j * rng.standard_normal((K, ng))
    M[517, 40] = 1.0 + 1j * value
    ev, ec = np.array([[-1.0]]), np.sort(rng.uniform(1, 20, (1, K)))
    got = run(torch_dev, M, ev, ec, [0.0])[0]
    bad = np.zeros((ng, ng), dtype=bool)
    bad[40, :] = bad[:, 40] = True
    assert np.array_equal(~np.isfinite(got.real), bad)
    off = bad & ~np.eye(ng, dtype=bool)
    assert not np.isfinite(got.imag[off]).any() and np.isfinite(got[~bad]).all()
