"""Sums of the K splits and the mirror below the diagonal, at the edges of their 32
wide tiles: real and complex, overwriting and accumulating, with the head's row and
column written separately; chi equal to its (conjugate) transpose to the last bit.

Bound.  Both sides sum 2 K products (complex) or K (real) per part: (2 K + 8) 2^-53
of the sum of magnitudes each, and one more rounding where chi is added to.
"""

import numpy as np
import pytest

import oracle
from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("flavor", ["real", "imag", "retarded"])
@pytest.mark.parametrize("ng", [1, 31, 32, 33, 65, 129, 1537])
def test_finalize(ng, flavor, accumulate):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(ng)
    nk, nv, nc = 2, 3, 37
    K = nk * nv * nc
    M = rng.standard_normal((K, ng))
    if flavor != "real":
        M = M + 1j * rng.standard_normal((K, ng))
    ev, ec = np.sort(rng.uniform(-10, 0, (nk, nv))), np.sort(rng.uniform(1, 20, (nk, nc)))
    om = np.array([0.0]) if flavor == "real" else np.array([0.0, 3.0])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    q = dict(M=dev(M), ev=dev(ev), ec=dev(ec), nk=nk, nv=nv, nc=nc, prefactor=0.5)
    old = rng.standard_normal((len(om), ng, ng)) + (0 if flavor == "real" else 1j)
    old = old + old.conj().transpose(0, 2, 1)
    chis = [dev(old)] if accumulate else None
    h = bgw.Handle(0)
    if flavor == "real":
        (chi,) = h.chi0_real([q], om, accumulate=accumulate, chis=chis)
        w = oracle.weights(ev, ec, om)
    elif flavor == "imag":
        (chi,) = h.chi0([dict(q, head=-1)], om, accumulate=accumulate, chis=chis)
        w = oracle.weights(ev, ec, om)
    else:
        (chi,) = h.chi0([dict(q, head=-1)], om, accumulate=accumulate, chis=chis, axis="retarded", broadening=0.3)
        w = oracle.weights_real(ev, ec, om, 0.3, "retarded")
    torch.cuda.synchronize()
    h.close()
    got = chi.cpu().numpy()
    size = np.abs(M.real) + np.abs(M.imag)
    for i in range(len(om)):
        wi = w[i].reshape(K, 1)
        ref = 0.5 * M.conj().T @ (wi * M) + (old[i] if accumulate else 0)
        mass = 0.5 * size.T @ ((np.abs(wi.real) + np.abs(wi.imag)) * size)
        bound = 2 * (2 * K + 8) * 2.0 ** -53 * (mass + (np.abs(old[i]) if accumulate else 0))
        assert np.all(np.abs(got[i] - ref) <= bound)
        if flavor != "retarded":
            assert np.array_equal(got[i], got[i].conj().T)
