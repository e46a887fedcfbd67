"""The split chi sum's workspace stays within what its first form took (BF16 digits: four
slices of 192 real rows, 2 bytes each, in columns padded to 128, one exponent of 4 bytes
per column and run of 96 pairs, and one byte more per weight vector), so that a limit set
to that still admits every call; results under it agree with those without."""

import numpy as np
import pytest

from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


def al(b):
    return (b + 255) // 256 * 256


def first_need(K, ng, vectors, partial, head):
    """K <= 96: one run, so one K split whatever the device."""
    pad = (ng + 127) // 128 * 128
    need = vectors * al(8 * (K + 128)) + al((4 * 192 * 2 + 4) * pad) + al(vectors * pad) + 256
    if partial:
        need += al(16 * vectors * ng * ng)
    if head:
        need += al(16 * 128 * vectors * ng)
    return need


@pytest.mark.parametrize("axis,nw,ng", [(axis, nw, ng) for axis, nw in (("imag", 1), ("imag", 32), ("retarded", 4), ("imag", 300))
                                        for ng in (1, 33, 96, 97, 100, 128, 129, 256, 257, 500, 1025) if nw * ng <= 40000])
@pytest.mark.parametrize("K", [1, 32, 95, 96])
def test_not_above_the_first_form(K, ng, axis, nw, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    gen = torch.Generator(device="cuda:0").manual_seed(ng)
    rnd = lambda *s, **k: torch.randn(*s, device="cuda:0", generator=gen, **k)  # noqa: E731
    q = dict(M=rnd(K, ng, dtype=torch.complex128), ev=-rnd(1, 1, dtype=torch.float64).abs(),
             ec=1.0 + rnd(1, K, dtype=torch.float64).abs().sort(1).values, nk=1, nv=1, nc=K, head=0, prefactor=0.5)
    kw = dict(precision=bgw.SPLIT_BF16, axis=axis, broadening=0.0 if axis == "imag" else 0.3)
    om = np.linspace(0.0, 20.0, nw)
    chis = [torch.empty((nw, ng, ng), dtype=torch.complex128, device="cuda:0")]
    limit = first_need(K, ng, nw * (1 if axis == "imag" else 2), axis != "imag", True)
    h = bgw.Handle(0)
    assert h.chi0_workspace([q], om, chis=chis, **kw) <= limit
    (a,) = h.chi0([q], om, **kw)
    h.close()
    monkeypatch.setenv("BGW_WORKSPACE_LIMIT", str(limit))
    h = bgw.Handle(0)
    (b,) = h.chi0([q], om, chis=chis, **kw)
    torch.cuda.synchronize()
    h.close()
    assert torch.equal(a, b)
