"""Error of epsilon^-1 without interchanges against the true inverse, on the symmetrised
scale, beside that of the elimination with partial pivoting of the same matrix.

The error is X (I - eps X), with the residual in twice the working precision: chi X from
20-bit pieces of both (their products of n <= 4096 terms are exact in 64 bits), v and
the differences with their rounding errors kept.

Bar.  Both add each sum of products once to what it changes, and on a matrix like this
neither grows: at most 3/2 of the pivoted one's.
"""

import numpy as np
import pytest

from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


def two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def halves(a):
    c = 134217729.0 * a
    hi = c - (c - a)
    return hi, a - hi


def two_prod(a, b):
    p = a * b
    (ah, al), (bh, bl) = halves(a), halves(b)
    return p, ((ah * bh - p) + ah * bl + al * bh) + al * bl


def pieces(torch, a, dim):
    e = torch.ceil(torch.log2(a.abs().amax(dim, keepdim=True).clamp_min(1e-300))) + 1
    out = []
    for k in range(4):
        q = torch.exp2(e - 20 * (k + 1))
        out.append(torch.round(a / q) * q)
        a = a - out[-1]
    return out


def product(torch, a, b):
    pa, pb = pieces(torch, a, 1), pieces(torch, b, 0)
    hi, lo = torch.zeros_like(a), torch.zeros_like(a)
    for p in range(5, -1, -1):
        for i in range(max(0, p - 3), min(p, 3) + 1):
            hi, e = two_sum(hi, pa[i] @ pb[p - i])
            lo += e
    return hi, lo


def error(torch, chi, v, x):
    n = len(v)
    cr, ci, xr, xi = (t.contiguous() for t in (chi.real, chi.imag, x.real, x.imag))
    eye = torch.eye(n, dtype=torch.float64, device=v.device)
    res = []
    for a, b, c, d, x0, one in ((cr, xr, -ci, xi, xr, eye), (cr, xi, ci, xr, xi, 0.0 * eye)):
        (h1, l1), (h2, l2) = product(torch, a, b), product(torch, c, d)
        h, e = two_sum(h1, h2)
        p, pe = two_prod(v[:, None].expand(n, n), h)
        s, e1 = two_sum(p, -x0)
        s, e2 = two_sum(s, one)
        res.append(s + (e1 + e2 + pe + v[:, None] * (l1 + l2 + e)))
    vs = torch.sqrt(v)
    scale = vs[None, :] / vs[:, None]
    err = x @ torch.complex(*res)
    return float(torch.linalg.matrix_norm(err * scale) / torch.linalg.matrix_norm(x * scale))


@pytest.mark.parametrize("n", [130, 700, 3100, 4000])
def test_error(n):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    env = torch.exp(-3.0 * torch.arange(n, dtype=torch.float64, device="cuda:0") / n)
    a = torch.randn(n, n, dtype=torch.complex128, device="cuda:0", generator=gen) * env
    chi = -0.3 * (a.mH @ a) / n
    chi = (0.5 * (chi + chi.mH))[None]
    v = 0.05 * 1000.0 ** torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen)
    v[0] = 1e4
    h = bgw.Handle(0)
    x, i1 = h.eps_inv(v, chi, nsd=True)
    p, i2 = h.eps_inv(v, chi)
    torch.cuda.synchronize()
    h.close()
    assert int(i1.abs().max()) == 0 and int(i2.abs().max()) == 0
    assert error(torch, chi[0], v, x[0]) <= 1.5 * error(torch, chi[0], v, p[0])
