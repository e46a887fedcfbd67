"""Timed workloads of the library, through its public entry points (paper_1111_4429_amd.bgw).

A case is one call, or one step of calls, of a polarizability calculation: pair densities, the chi sum, the
inverse dielectric matrix, and the self-energy and real-flavor paths that run on the same kernels.  The sizes are
those of the synthetic workloads (paper_1111_4429_amd/synth.py), with fewer pairs or frequencies where one pass of
the whole workload takes seconds; ``draw`` spreads the same kinds of calls over the same ranges.

All inputs are drawn on the GPU from the seed.  ``exact`` is plain torch in 64 bits.
"""

import math

import numpy as np
import torch

from paper_1111_4429_amd import bgw

HARTREE_EV = 27.211386245988
DEV = "cuda:0"
_HANDLE = None


def _handle():
    """The one handle per device that a program keeps."""
    global _HANDLE
    if _HANDLE is None:
        _HANDLE = bgw.Handle(0)
    return _HANDLE


def listed():
    return [
        # the smallest whole step (16^3 grid): pair densities, static chi, eps^-1; launches and host work count
        dict(name="step-tiny-16", kind="step", n=16, ngw=300, ng=300, nk=1, nv=4, nc=16),
        # pair densities of a small cell with many k-points, 24^3 transform box
        dict(name="pair-silicon-48", kind="pair", n=48, ngw=1500, ng=1500, nk=64, nv=4, nc=400),
        # pair densities of a medium cell at one k-point, many valence bands, 32^3 box
        dict(name="pair-medium-64", kind="pair", n=64, ngw=4000, ng=4000, nk=1, nv=64, nc=128),
        # pair densities of one q with large spheres and odd counts, 48^3 box
        dict(name="pair-sphere-6000", kind="pair", n=48, ngw=6000, ng=5501, nk=1, nv=32, nc=151),
        # static chi sum of the small cell in FP64
        dict(name="chi-fp64-1500", kind="chi", precision="fp64", axis="imag", ng=1500, ng2=0, nk=64, nv=4, nc=400,
             nw=1, emax=0.0),
        # chi sum of the medium cell at imaginary frequencies, split precision
        dict(name="chi-split-4000", kind="chi", precision="split", axis="imag", ng=4000, ng2=0, nk=8, nv=8, nc=640,
             nw=4, emax=100.0),
        # retarded chi on real frequencies of two q with uneven spheres in one call, split precision
        dict(name="chi-split-retarded", kind="chi", precision="split", axis="retarded", ng=1500, ng2=731, nk=16,
             nv=4, nc=400, nw=6, emax=30.0),
        # eps^-1 of one static matrix, small cell
        dict(name="eps-nsd-1500", kind="eps", general=False, ng=1500, nw=1),
        # eps^-1 at several imaginary frequencies, medium cell
        dict(name="eps-nsd-4000x4", kind="eps", general=False, ng=4000, nw=4),
        # eps^-1 at several real frequencies (general matrices, partial pivoting)
        dict(name="eps-pivot-1500x8", kind="eps", general=True, ng=1500, nw=8),
        # static self-energy of one q: bare exchange, screened exchange, Coulomb hole
        dict(name="sigma-48", kind="sigma", nocc=4, ninner=404, nouter=64, ng=1500),
        # real flavor: real pair densities, then the real static chi
        dict(name="real-48", kind="real", n=48, ngw=1500, ng=1500, nk=16, nv=4, nc=400),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "pair", "pair", "pair", "chi", "chi", "chi", "eps", "eps", "sigma", "real"])
    if kind in ("step", "pair", "real"):
        small = kind == "step"
        ngw = _log(rng, 60, 300) if small else _log(rng, 150, 2500 if kind == "real" else 6000)
        ng = min(ngw, _log(rng, 40, ngw))
        n = 16 if ngw <= 300 else 48 if rng.random() < 0.7 else 64
        nv = rng.randint(2, 6) if small else _log(rng, 2, 48)
        nc = min(ngw // 3, _log(rng, 5, 40) if small else _log(rng, 16, 400))
        # pairs: at most about the pair work of the listed cases (points of the transform grid per pair)
        most = 300 if small else int(min(8.0e8 / ngw ** 1.25, 1.2e8 / ng))
        nk = max(1, min(_log(rng, 1, 2 if small else 32), most // (nv * nc)))
        nv = max(1, min(nv, most // (nk * nc)))
        return dict(kind=kind, n=n, ngw=ngw, ng=ng, nk=nk, nv=nv, nc=nc)
    if kind == "chi":
        precision = rng.choice(["fp64", "split"])
        axis = rng.choice(["imag", "imag", "retarded", "advanced"])
        ng = _log(rng, 150, 4000)
        ng2 = rng.choice([0, max(100, int(ng * rng.uniform(0.3, 0.95)))])
        nw = rng.choice([1, 1, 2, 4, 6])
        emax = 0.0 if nw == 1 and axis == "imag" else rng.uniform(10.0, 60.0)
        vectors = nw * (1 if axis == "imag" else 2)
        cost = 4.0 * (ng * ng + ng2 * ng2) * vectors
        K = min(_log(rng, 1500, 80000), int((0.9e12 if precision == "fp64" else 8.0e12) / cost), int(1.2e8 / (ng + ng2)))
        nv = rng.randint(2, 8)
        nc = _log(rng, 20, 400)
        nk = max(1, K // (nv * nc))
        return dict(kind="chi", precision=precision, axis=axis, ng=ng, ng2=ng2, nk=nk, nv=nv, nc=nc, nw=nw, emax=emax)
    if kind == "eps":
        general = rng.random() < 0.4
        ng = _log(rng, 100, 2200 if general else 4000)
        return dict(kind="eps", general=general, ng=ng, nw=max(1, min(rng.choice([1, 2, 4, 8]), int(2.4e11 / ng ** 3))))
    ng, ninner = _log(rng, 200, 1500), _log(rng, 20, 404)
    return dict(kind="sigma", nocc=max(1, ninner // 10), ninner=ninner, nouter=_log(rng, 6, 64), ng=ng)


# ---------------------------------------------------------------- inputs


def _sphere(count):
    """The first `count` Miller triples by (m.m, m_x, m_y, m_z)."""
    r = int((count / 4.0) ** (1.0 / 3.0)) + 4
    ax = np.arange(-r, r + 1)
    m = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    order = np.lexsort((m[:, 2], m[:, 1], m[:, 0], (m * m).sum(1)))
    return np.ascontiguousarray(m[order[:count]].astype(np.int32))


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _norm2(g):
    return torch.from_numpy((g.astype(np.float64) ** 2).sum(1)).to(DEV)


def _randn(gen, shape, real=False):
    if real:
        return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, device=DEV, dtype=torch.float64))


def _bands(gen, nk, nb, gw, real=False):
    """nk sets of nb orthonormal plane-wave states with a Gaussian envelope."""
    c = _randn(gen, (nk, nb, len(gw)), real) * torch.exp(-_norm2(gw) / 16.0)
    for k in range(nk):
        low = torch.linalg.cholesky(c[k] @ c[k].conj().T)
        c[k] = torch.linalg.solve_triangular(low, c[k].clone(), upper=False)
    return c


def _energies(gen, nk, nv, nc):
    ev = torch.rand((nk, nv), generator=gen, device=DEV, dtype=torch.float64) * 10.0 - 10.0
    ec = torch.rand((nk, nc), generator=gen, device=DEV, dtype=torch.float64) * 19.0 + 1.0
    return ev.sort(1).values.contiguous(), ec.sort(1).values.contiguous()


def _pairs_g(gen, count, g):
    """Pair densities as the chi sum meets them: decaying with |G|, the G = 0 column of order |q0|."""
    m = _randn(gen, (count, len(g))) * (0.05 * torch.exp(-_norm2(g) / 32.0))
    m[:, 0] *= 1.0e-3
    return m


def _vcoul(g, nv=4, q0=1.0e-3):
    b = 2.0 * math.pi / (67.5 * nv) ** (1.0 / 3.0)
    m = torch.from_numpy(g.astype(np.float64)).to(DEV)
    m[:, 0] += q0
    return 4.0 * math.pi / (b * b * (m * m).sum(1))


def _omega(c):
    if c["nw"] == 1:
        return np.array([c["emax"]])
    if c["axis"] == "imag":  # Gauss-Legendre nodes on [0, emax] eV
        return 0.5 * c["emax"] * (np.polynomial.legendre.leggauss(c["nw"])[0] + 1.0)
    return np.linspace(0.0, c["emax"], c["nw"])


def _prefactor(c):
    return 1.0 / (c["nk"] * 67.5 * c["nv"])


BROADENING = 0.1  # eV, real axis


def _states(c, seed):
    gen = _gen(seed)
    real = c["kind"] == "real"
    gw, ge = _sphere(c["ngw"]), _sphere(c["ng"])
    cc = _bands(gen, c["nk"], c["nc"], gw, real)
    cv = _bands(gen, c["nk"], c["nv"], gw, real)
    ev, ec = _energies(gen, c["nk"], c["nv"], c["nc"])
    return dict(gw=gw, ge=ge, cv=cv, cc=cc, ev=ev, ec=ec, v=_vcoul(ge, c["nv"]))


def _chi_inputs(c, seed):
    gen = _gen(seed)
    qs = []
    for ng in [c["ng"]] + ([c["ng2"]] if c["ng2"] else []):
        ev, ec = _energies(gen, c["nk"], c["nv"], c["nc"])
        qs.append(dict(M=_pairs_g(gen, c["nk"] * c["nv"] * c["nc"], _sphere(ng)), ev=ev, ec=ec, nk=c["nk"], nv=c["nv"],
                       nc=c["nc"], head=0, prefactor=_prefactor(c)))
    return qs


def _eps_inputs(c, seed):
    gen = _gen(seed)
    g = _sphere(c["ng"])
    rank = max(8, c["ng"] // 2)
    env = torch.exp(-_norm2(g) / 32.0)
    env[0] = 1.0e-3
    chi = torch.empty((c["nw"], c["ng"], c["ng"]), dtype=torch.complex128, device=DEV)
    for w in range(c["nw"]):
        a = _randn(gen, (rank, c["ng"])) * env
        h = (a.conj().T @ a) * (-0.15 / (rank * (1.0 + w)))
        chi[w] = 0.5 * (h + h.conj().T)
        if c["general"]:  # retarded: an anti-Hermitian part beside the Hermitian one
            a = _randn(gen, (rank, c["ng"])) * env
            h = (a.conj().T @ a) * (-0.1 / rank)
            chi[w] += 0.5j * (h + h.conj().T)
    return dict(chi=chi, v=_vcoul(g))


def _sigma_inputs(c, seed):
    gen = _gen(seed)
    g = _sphere(c["ng"])
    m = _pairs_g(gen, c["ninner"] * c["nouter"], g).reshape(c["ninner"], c["nouter"], c["ng"])
    einv = _randn(gen, (c["ng"], c["ng"])) * 0.01
    einv.diagonal().add_(1.0)
    return dict(M=m, Mocc=m[:c["nocc"]].contiguous(), v=_vcoul(g, q0=0.05), einv=einv)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, h=_handle())
    if kind in ("step", "pair", "real"):
        s.update(_states(case, seed))
    elif kind == "chi":
        s["qs"] = _chi_inputs(case, seed)
        s["omega"] = _omega(case)
    elif kind == "eps":
        s.update(_eps_inputs(case, seed))
    else:
        s.update(_sigma_inputs(case, seed))
    return s


# ---------------------------------------------------------------- one pass


def run(s):
    c, h = s["case"], s["h"]
    kind = c["kind"]
    if kind == "chi":
        return h.chi0(s["qs"], s["omega"], precision=bgw.SPLIT_BF16 if c["precision"] == "split" else bgw.FP64,
                      axis=c["axis"], broadening=0.0 if c["axis"] == "imag" else BROADENING)
    if kind == "eps":
        return h.eps_inv(s["v"], s["chi"], nsd=not c["general"])
    if kind == "sigma":
        return [h.sigma("x", s["Mocc"], s["v"], 0.01, head=0),
                h.sigma("sx", s["Mocc"], s["v"], 0.01, epsinv=s["einv"]),
                h.sigma("ch", s["M"], s["v"], 0.01, epsinv=s["einv"])]
    if kind == "pair":
        return h.pair_density(c["n"], s["gw"], s["ge"], s["cv"], s["cc"])
    q = dict(ev=s["ev"], ec=s["ec"], nk=c["nk"], nv=c["nv"], nc=c["nc"], head=0, prefactor=_prefactor(c))
    if kind == "real":
        m = h.pair_density_real(c["n"], s["gw"], s["ge"], s["cv"], s["cc"])
        return m, h.chi0_real([dict(q, M=m)], [0.0])[0]
    m = h.pair_density(c["n"], s["gw"], s["ge"], s["cv"], s["cc"])
    chi = h.chi0([dict(q, M=m)], [0.0])[0]
    return m, chi, h.eps_inv(s["v"], chi, nsd=True)


# ---------------------------------------------------------------- what a pass cannot do without


def _box(c):
    """Side of the smallest alias-free cube of the transforms."""
    return 2 * int(np.abs(_sphere(c["ngw"])).max()) + int(np.abs(_sphere(c["ng"])).max()) + 1


def work(case):
    c, kind = case, case["kind"]
    size = 8 if kind == "real" else 16
    if kind in ("step", "pair", "real"):
        K, n3 = c["nk"] * c["nv"] * c["nc"], _box(c) ** 3
        bands = c["nk"] * (c["nv"] + c["nc"])
        fft = 5.0 * n3 * math.log2(n3) * (0.5 if kind == "real" else 1.0)
        out = dict(bytes=size * (bands * c["ngw"] + K * c["ng"]), flops=bands * fft + K * (fft + 6.0 * n3))
        if kind == "step":
            out["bytes"] += 16 * (K * c["ng"] + 3 * c["ng"] ** 2)
            out["flops"] += 4.0 * c["ng"] ** 2 * K + 8.0 * c["ng"] ** 3
        if kind == "real":
            out["bytes"] += 8 * (K * c["ng"] + c["ng"] ** 2)
            out["flops"] += 1.0 * c["ng"] ** 2 * K
        return out
    if kind == "chi":
        K = c["nk"] * c["nv"] * c["nc"]
        vectors = c["nw"] * (1 if c["axis"] == "imag" else 2)
        n1, n2 = c["ng"] + c["ng2"], c["ng"] ** 2 + c["ng2"] ** 2
        return dict(bytes=16 * (K * n1 + c["nw"] * n2), flops=4.0 * n2 * K * vectors)
    if kind == "eps":
        return dict(bytes=32 * c["nw"] * c["ng"] ** 2, flops=8.0 * c["nw"] * c["ng"] ** 3)
    ng, no = c["ng"], c["nouter"]
    screened = sum(8.0 * ni * no * ng * (ng + no) for ni in (c["nocc"], c["ninner"]))
    return dict(bytes=16 * ((c["ninner"] + 2 * c["nocc"]) * no * ng + 2 * ng * ng + 3 * no * no),
                flops=screened + 4.0 * no * no * ng * c["nocc"])


# ---------------------------------------------------------------- the same results from plain torch in 64 bits


def _exact_pairs(c, s):
    n = _box(c)
    n += n % 2
    gw, ge = (torch.from_numpy(g.astype(np.int64)).to(DEV) % n for g in (s["gw"], s["ge"]))
    iw, ie = ((g[:, 0] * n + g[:, 1]) * n + g[:, 2] for g in (gw, ge))

    def real_space(coeff):
        grid = torch.zeros((coeff.shape[0], n ** 3), dtype=torch.complex128, device=DEV)
        grid[:, iw] = coeff.to(torch.complex128)
        return torch.fft.ifftn(grid.view(-1, n, n, n), dim=(1, 2, 3), norm="forward")

    out = torch.empty((c["nk"], c["nv"], c["nc"], len(ie)), dtype=torch.complex128, device=DEV)
    step = max(1, int(2.0e9 / (16 * n ** 3)))
    for k in range(c["nk"]):
        uv = real_space(s["cv"][k])
        for c0 in range(0, c["nc"], step):
            uc = real_space(s["cc"][k, c0:c0 + step])
            for v in range(c["nv"]):
                p = torch.fft.ifftn(uv[v].conj() * uc, dim=(1, 2, 3), norm="backward")
                out[k, v, c0:c0 + step] = p.reshape(p.shape[0], -1)[:, ie]
    return out.reshape(-1, len(ie))


def _exact_chi(m, ev, ec, prefactor, omega, axis):
    nk, nv = ev.shape
    d = ((ev[:, :, None] - ec[:, None, :]) / HARTREE_EV).reshape(-1)
    mh = m.conj().T
    out = []
    for x in omega:
        e, dl = float(x) / HARTREE_EV, BROADENING / HARTREE_EV * (-1.0 if axis == "advanced" else 1.0)
        if axis == "imag":
            w = d / (d * d + e * e)
        else:
            w = 0.5 * (1.0 / torch.complex(d - e, torch.full_like(d, -dl)) + 1.0 / torch.complex(d + e, torch.full_like(d, dl)))
        acc = torch.zeros((m.shape[1], m.shape[1]), dtype=m.dtype, device=DEV)
        for t in range(0, m.shape[0], 16384):
            acc += mh[:, t:t + 16384] @ (w[t:t + 16384, None] * m[t:t + 16384])
        out.append(prefactor * acc)
    return torch.stack(out)


def _exact_eps(chi, v):
    chi, v = chi.cpu(), v.cpu()  # LAPACK on the host: seconds at ng = 4000
    eye = torch.eye(chi.shape[1], dtype=chi.dtype)
    return torch.stack([torch.linalg.inv(eye - v[:, None] * x) for x in chi])


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "chi":
        return [_exact_chi(q["M"], q["ev"], q["ec"], q["prefactor"], _omega(c), c["axis"]) for q in _chi_inputs(c, seed)]
    if kind == "eps":
        s = _eps_inputs(c, seed)
        return _exact_eps(s["chi"], s["v"]), None
    if kind == "sigma":
        s = _sigma_inputs(c, seed)

        def contract(m, y):  # sum over (inner, G) of conj(m[i][n][G]) y[i][n'][G]
            a, b = (x.permute(1, 0, 2).reshape(c["nouter"], -1) for x in (m, y))
            return a.conj() @ b.T

        def screen(m, w):
            return (m.reshape(-1, c["ng"]) @ w.T).reshape(m.shape)

        vx = s["v"].clone()
        vx[0] = 0.0
        w = s["einv"] * s["v"]
        wc = w - torch.diag(s["v"]).to(w.dtype)
        return [-0.01 * contract(s["Mocc"], s["Mocc"] * vx), -0.01 * contract(s["Mocc"], screen(s["Mocc"], w)),
                0.005 * contract(s["M"], screen(s["M"], wc))]
    s = _states(c, seed)
    m = _exact_pairs(c, s)
    if kind == "pair":
        return m
    if kind == "real":
        m = m.real.contiguous()
        return m, _exact_chi(m, s["ev"], s["ec"], _prefactor(c), [0.0], "imag")
    chi = _exact_chi(m, s["ev"], s["ec"], _prefactor(c), [0.0], "imag")
    return m, chi, (_exact_eps(chi, s["v"]), None)
