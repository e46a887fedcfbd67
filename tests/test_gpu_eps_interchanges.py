"""Row interchanges of the pivoted epsilon^-1 in outer blocks of 64 (n < 3000) and 128
rows: pivots from inside the block, from outside it, and chains through the same row.

eps is a matrix dominated by its diagonal with its rows in another order, so that the
pivots are the rows of that order, or a random dense one.

Bound.  As for the other rank updates, a residual of at most 16 n 2^-53 |A| |X|, on the
dense ones times the growth that partial pivoting shows on such matrices, n^(2/3).
"""

import numpy as np
import pytest

from paper_1111_4429_amd import bgw

pytestmark = pytest.mark.gpu


def order(rng, n, form):
    p = np.arange(n)
    if form == "anywhere":
        rng.shuffle(p)
    elif form == "inside":  # every 128 rows among themselves, so inside their outer block
        for k in range(0, n, 128):
            rng.shuffle(p[k:k + 128])
    elif form == "outside":  # every row trades with one far below
        p = p[::-1].copy()
    elif form == "chain":  # the row of every pivot is the one that the pivot before it displaced
        p = np.roll(p, 1)
    else:  # both: the first half of every 128 rows inside, the second anywhere
        for k in range(0, n, 128):
            rng.shuffle(p[k:k + 64])
        rest = np.concatenate([np.arange(k + 64, min(n, k + 128)) for k in range(0, n, 128)])
        p[rest] = p[rng.permutation(rest)]
    return p


def interchanges(p):
    """Rows that change places when pivot j is the row that p puts at j."""
    at = np.argsort(p)  # row of pivot j
    where, holds, count = np.arange(len(p)), np.arange(len(p)), 0
    for j in range(len(p)):
        a, b = holds[j], at[j]
        if a != b:
            count += 1
            holds[where[b]], where[a] = a, where[b]
            holds[j], where[b] = b, j
    return count


@pytest.mark.parametrize("form", ["anywhere", "inside", "outside", "chain", "both", "dense"])
@pytest.mark.parametrize("n,nw", [(129, 3), (449, 2), (1537, 1), (3009, 2), (3072, 1), (3136, 1)])
def test_interchanges(n, nw, form):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(n)
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    eps = torch.randn(nw, n, n, dtype=torch.complex128, device="cuda:0", generator=gen)
    if form != "dense":
        eps *= 0.2 / np.sqrt(n)
        eye = torch.eye(n, dtype=torch.float64, device="cuda:0")
        eps += eye * (1.0 + torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen))
        for w in range(nw):
            p = order(rng, n, form)
            assert interchanges(p) >= n // 4
            eps[w] = eps[w][torch.from_numpy(p).to("cuda:0")]
    one = torch.ones(n, dtype=torch.float64, device="cuda:0")
    eye = torch.eye(n, dtype=eps.dtype, device="cuda:0")
    h = bgw.Handle(0)
    inv, info = h.eps_inv(one, eye - eps)
    torch.cuda.synchronize()
    h.close()
    assert int(info.abs().max()) == 0
    grow = n ** (2.0 / 3.0) if form == "dense" else 1.0
    for w in range(nw):
        a = eye - (eye - eps[w])  # what the library is given, to the last bit
        bound = 16 * n * 2.0 ** -53 * grow * torch.linalg.matrix_norm(a) * torch.linalg.matrix_norm(inv[w])
        assert float(torch.linalg.matrix_norm(a @ inv[w] - eye)) <= float(bound)
        if form != "dense":  # well-conditioned: close to the inverse of the same rows in their own order
            assert float(torch.linalg.matrix_norm(a @ inv[w] - eye)) <= 1e-12 * np.sqrt(n)
