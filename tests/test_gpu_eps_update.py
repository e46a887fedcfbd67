"""Rank updates of epsilon^-1 at the edges of their 32 and 64 wide tiles and of the
panels, with and without interchanges.

Bound.  Elimination of n columns leaves a residual of at most a small multiple of
n 2^-53 |A| |X| (no growth to speak of on these matrices); 16 is taken.
"""

import numpy as np
import pytest

from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsd", [True, False])
@pytest.mark.parametrize("n,nw", [(1, 1), (15, 2), (31, 1), (33, 3), (63, 2), (65, 1), (97, 2), (127, 1), (191, 3),
                                  (449, 41), (3009, 1)])
def test_edges(n, nw, nsd):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda:0", generator=gen)  # noqa: E731
    x = rnd(nw, n, n)
    chi = -(x @ x.mH) / n
    chi = 0.5 * (chi + chi.mH)
    if not nsd:
        chi = chi + 0.3 * rnd(nw, n, n) / np.sqrt(n)
    v = torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen) + 0.5
    h = bgw.Handle(0)
    inv, info = h.eps_inv(v, chi, nsd=nsd)
    torch.cuda.synchronize()
    h.close()
    assert int(info.abs().max()) == 0
    eye = torch.eye(n, dtype=chi.dtype, device="cuda:0")
    for w in range(nw):
        a = eye - v[:, None] * chi[w]
        res = torch.linalg.matrix_norm(a @ inv[w] - eye)
        bound = 16 * n * 2.0 ** -53 * torch.linalg.matrix_norm(a) * torch.linalg.matrix_norm(inv[w])
        assert float(res) <= float(bound)
