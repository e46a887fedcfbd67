"""Rank updates of epsilon^-1 at the edges of their 32 and 64 wide tiles and of the
panels, with and without interchanges.

Bound.  Elimination of n columns leaves a residual of at most a small multiple of
n 2^-53 |A| |X| (no growth to speak of on these matrices); 16 is taken.  Without
interchanges that holds on the symmetrised scale, v^-1/2 (.) v^1/2.
"""

import numpy as np
import pytest

from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


SIZES = [(1, 1), (15, 2), (17, 1), (31, 1), (33, 3), (49, 1), (63, 2), (65, 1), (97, 2), (127, 1), (191, 3), (449, 41),
         (3009, 1), (3010, 2), (3072, 1), (3136, 1)]


# "hermitian": exactly, so eliminated by its upper triangle; "nearly": to 1e-10, as a
# general matrix, but without interchanges; "general": with interchanges; "mixed": the
# first two in one call
@pytest.mark.parametrize("form", ["hermitian", "nearly", "mixed", "general"])
@pytest.mark.parametrize("n,nw", SIZES)
def test_edges(n, nw, form):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda:0", generator=gen)  # noqa: E731
    x = rnd(nw, n, n)
    chi = -(x @ x.mH) / n
    chi = 0.5 * (chi + chi.mH)
    if form == "general":
        chi = chi + 0.3 * rnd(nw, n, n) / np.sqrt(n)
    if form == "nearly":
        chi = chi + 1e-10 * rnd(nw, n, n)
    if form == "mixed":
        chi[::2] += 1e-10 * rnd((nw + 1) // 2, n, n)
    v = 50.0 ** torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen) / 10.0
    h = bgw.Handle(0)
    inv, info = h.eps_inv(v, chi, nsd=form != "general")
    torch.cuda.synchronize()
    h.close()
    assert int(info.abs().max()) == 0
    eye = torch.eye(n, dtype=chi.dtype, device="cuda:0")
    vs = torch.sqrt(v) if form != "general" else torch.ones_like(v)
    for w in range(nw):
        a = (eye - v[:, None] * chi[w]) * vs[None, :] / vs[:, None]
        x = inv[w] * vs[None, :] / vs[:, None]
        res = torch.linalg.matrix_norm(a @ x - eye)
        bound = 16 * n * 2.0 ** -53 * torch.linalg.matrix_norm(a) * torch.linalg.matrix_norm(x)
        assert float(res) <= float(bound)
