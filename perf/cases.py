"""Measured cases of the library: the calls that a GW program makes, over the range of their sizes.

A case names one call (kind) and its sizes:
  build    gw_chi0_build: chi0 of nq q-points at nomega frequencies, nv valence states x ncol columns
           (the last `windows` of them window representatives with a multiplicity);
  adjoint  gw_chi0_backward of such a build: the energy and multiplicity gradients, with coef the
           coefficient gradients too;
  inverse  gw_eps_inv of nbatch matrices, static (hermitian) or dynamic;
  coh      gw_sigma_coh_static, nv states x ncol columns;
  gpp      gw_sigma_coh_gpp, the same at nenergy energies.
Spheres, energies and cells are the generator's shapes (simple-cubic cells, wavefunction sphere of a
quarter of the grid, dielectric sphere ordered by |q+G|, valence energies in [-10, 0] eV, conduction
energies with density sqrt(E) on [5, 60] eV, orthonormal random coefficients).
"""
import math
from functools import lru_cache

import numpy as np
import torch

import paper_1601_06767_amd as gw

EV = 1.0 / 27.211386245988
QS = [(0.01, 0.0, 0.0), (0.5, 0.0, 0.0), (0.0, 0.5, 0.0), (0.5, 0.5, 0.0)]
C128 = torch.complex128


def listed():
    return [
        # the smallest call: a 2-atom-sized cell in full, where launches and latency count
        {"name": "build 24 fp64", "kind": "build", "nd": 24, "nv": 16, "ncol": 240, "ng": 259, "prec": "fp64",
         "nomega": 1, "nq": 1, "windows": 0},
        # the 64-atom cell, static: four conduction chunks in double precision
        {"name": "build 72 fp64", "kind": "build", "nd": 72, "nv": 128, "ncol": 1000, "ng": 2000, "prec": "fp64",
         "nomega": 1, "nq": 1, "windows": 0},
        # the same cell in the mixed precision, all 4000 bands
        {"name": "build 72 bf16x3", "kind": "build", "nd": 72, "nv": 128, "ncol": 4000, "ng": 2000,
         "prec": "bf16x3", "nomega": 1, "nq": 1, "windows": 0},
        # the 128-atom cell, explicit bands and energy windows
        {"name": "build 96 grouped bf16x3", "kind": "build", "nd": 96, "nv": 256, "ncol": 900, "ng": 4000,
         "prec": "bf16x3", "nomega": 1, "nq": 1, "windows": 30},
        # the 256-atom cell, a share of its columns (the largest spheres)
        {"name": "build 128 grouped bf16x3", "kind": "build", "nd": 128, "nv": 512, "ncol": 318, "ng": 8000,
         "prec": "bf16x3", "nomega": 1, "nq": 1, "windows": 30},
        # several q-points with their own spheres, several frequencies with broadening
        {"name": "build 72 batched fp32", "kind": "build", "nd": 72, "nv": 128, "ncol": 250, "ng": 1429,
         "prec": "fp32", "nomega": 4, "nq": 3, "windows": 0},
        # gradients for band energies, window weights and wavefunctions, double precision
        {"name": "adjoint 72 coef fp64", "kind": "adjoint", "nd": 72, "nv": 64, "ncol": 250, "ng": 2000,
         "prec": "fp64", "nomega": 1, "nq": 1, "windows": 0, "coef": True},
        # gradients for energies in the mixed precision, grouped columns
        {"name": "adjoint 96 grouped bf16x3", "kind": "adjoint", "nd": 96, "nv": 256, "ncol": 250, "ng": 4000,
         "prec": "bf16x3", "nomega": 1, "nq": 1, "windows": 30, "coef": False},
        # the dielectric inverse behind every static chi0
        {"name": "inverse static 2000", "kind": "inverse", "ng": 2000, "nbatch": 1, "hermitian": True},
        # and behind a set of frequencies
        {"name": "inverse dynamic 4x1114", "kind": "inverse", "ng": 1114, "nbatch": 4, "hermitian": False},
        # self-energy of the band-edge states over bands: static limit and plasmon pole
        {"name": "coh 72", "kind": "coh", "nd": 72, "nv": 8, "ncol": 2000, "ng": 2000, "windows": 0},
        {"name": "gpp 72", "kind": "gpp", "nd": 72, "nv": 8, "ncol": 300, "ng": 800, "windows": 20, "nenergy": 4},
    ]


def _ng_of(nd):
    return 8000.0 * (nd / 128.0) ** 2.4


def _seconds(c):
    """Rough cost of a case, to keep drawn ones within the largest listed one."""
    if c["kind"] == "inverse":
        return c["nbatch"] * (c["ng"] * 7e-6 + 8.0 * c["ng"] ** 3 / 30e12)
    pairs = float(c["nv"] * c["ncol"] * c.get("nq", 1))
    prec = c.get("prec", "fp64")
    t = (pairs + 40 * (c["nv"] + c["ncol"])) * c["nd"] ** 3 * (4e-12 if prec == "fp64" else 2e-12)
    rate = {"fp64": 50e12, "fp32": 100e12, "bf16x3": 250e12}[prec]
    t += pairs * c["ng"] ** 2 * c.get("nomega", 1) * (16 if c.get("nomega", 1) > 1 else 4) / rate
    if c["kind"] == "adjoint":
        t = 3 * t + (3 * t if c["coef"] else 0)
    if c["kind"] == "gpp":
        t += c["ncol"] * c["nenergy"] * ((c["nv"] + 7) // 8) ** 2 * c["ng"] ** 2 * 150 / 20e12
    return t


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build"] * 6 + ["adjoint"] * 2 + ["inverse"] * 2 + ["coh", "gpp"])
    if kind == "inverse":
        herm = rng.random() < 0.5
        nb = rng.choice([1, 1, 2, 3, 4])
        return {"kind": kind, "ng": _log(rng, 200, 6000 if herm and nb == 1 else 2500), "nbatch": nb, "hermitian": herm}
    nd = rng.choice([24, 48, 64, 72, 72, 96, 96, 128, 40, 56, 80])
    c = {"kind": kind, "nd": nd, "ng": min(8000, int(_ng_of(nd) * rng.uniform(0.35, 1.05)) + 90)}
    if kind in ("coh", "gpp"):
        c["nv"] = rng.randint(2, 16 if kind == "coh" else 9)
        c["ncol"] = _log(rng, 60, 4000 if kind == "coh" else 500)
        if kind == "gpp":
            c["ng"] = min(c["ng"], 1500)
            c["nenergy"] = rng.randint(1, 9)
    else:
        c["prec"] = rng.choice(["fp64", "fp32", "bf16x3", "bf16x3"])
        c["nv"] = _log(rng, 8, 512)
        c["ncol"] = _log(rng, 40, 3000)
        many = kind == "build" and rng.random() < 0.35
        c["nomega"] = rng.randint(2, 6) if many else 1
        c["nq"] = rng.randint(1, 3) if many else 1
        if kind == "adjoint":
            c["coef"] = c["prec"] == "fp64" and nd in (24, 72) and rng.random() < 0.6
            if c["coef"]:   # spheres that the gradients' kernels are built for
                c["ng"] = rng.randint(110, 500) if nd == 24 else rng.randint(500, 2100)
    c["windows"] = rng.choice([0, 0, 7, 30])
    while _seconds(c) > 0.3 and (c["ncol"] > 45 or c["nv"] > 8):
        k = "ncol" if c["ncol"] > 45 else "nv"
        c[k] = max(40 if k == "ncol" else 5, int(c[k] * 0.8))
    c["windows"] = min(c["windows"], c["ncol"] // 4)
    return c


# ---------------------------------------------------------------- inputs
@lru_cache(maxsize=None)
def _wf_sphere(nd):
    r = nd // 4
    a = np.arange(-r, r + 1)
    g = np.stack(np.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    k = (g * g).sum(1)
    g, k = g[k <= r * r], k[k <= r * r]
    return np.ascontiguousarray(g[np.lexsort((g[:, 2], g[:, 1], g[:, 0], k))].astype(np.int32))


@lru_cache(maxsize=None)
def _chi_sphere(ng, q):
    r = int((ng * 3.0 / (4.0 * math.pi)) ** (1.0 / 3.0)) + 3
    a = np.arange(-r, r + 1)
    g = np.stack(np.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    k = np.round(((g + np.array(q)) ** 2).sum(1), 9)
    return np.ascontiguousarray(g[np.lexsort((g[:, 2], g[:, 1], g[:, 0], k))[:ng]].astype(np.int32))


def _lattice(nd):
    """Simple-cubic constant (bohr) of the cell whose grid this is (8.4 bohr at 24, 16.8 at 72 ...)."""
    return 8.4 * {24: 1.0, 72: 2.0, 96: 16 ** (1 / 3), 128: 32 ** (1 / 3)}.get(nd, nd / 38.0)


def _coulomb(a, g, q):
    k2 = (((g + np.array(q)) * (2.0 * math.pi / a)) ** 2).sum(1)
    return 2.0 / a ** 3 * 4.0 * math.pi / k2


def _orthonormal(gen, n, npw):
    x = torch.randn((n, npw), generator=gen, device="cuda", dtype=C128)
    lo = torch.linalg.cholesky(x @ x.conj().T)
    eye = torch.eye(n, device="cuda", dtype=C128)
    inv = [torch.linalg.solve_triangular(lo, eye[:, k:k + 256].contiguous(), upper=False) for k in range(0, n, 256)]
    return torch.cat(inv, 1) @ x


class _Geometry:
    """Owns a context and its geometries; they go with the last reference."""

    def __init__(self):
        self.ctx = gw.gw_ctx_create(0)
        self.geoms = []

    def add(self, nd, wf, chi, a, q):
        g = gw.gw_geom_create(self.ctx, (nd,) * 3, wf, chi, np.eye(3) * a, q)
        self.geoms.append(g)
        return g

    def __del__(self):
        torch.cuda.synchronize()
        for g in self.geoms:
            gw.gw_geom_destroy(g)
        gw.gw_ctx_destroy(self.ctx)


def _ngs(case):
    """Sphere sizes of the q-points: uneven, up to the case's."""
    return [int(case["ng"] * (1.0 - 0.22 * i)) for i in range(case.get("nq", 1))]


def _omegas(case):
    n = case.get("nomega", 1)
    return [40.0 * EV * j / max(n, 2) for j in range(n)], (0.1 * EV if n > 1 else 0.0)


def _bands(case, gen, npw):
    """(coef_v, e_v, coef_c, e_col, n_col, col_band) of each q-point, on the GPU."""
    nv, nc, nw = case["nv"], case["ncol"], case["windows"]
    probs = []
    rows = _orthonormal(gen, nv + nc, npw) if nv + nc <= npw else None
    for iq in range(case.get("nq", 1)):
        if rows is None:   # more bands than plane waves (tiny cells): two sets of their own
            cv = _orthonormal(gen, nv, npw)
            cc = torch.randn((nc, npw), generator=gen, device="cuda", dtype=C128) / math.sqrt(npw)
        else:
            cv = rows[:nv] if iq == 0 else _orthonormal(gen, nv, npw)
            cc = rows[nv:]
        u = torch.rand(nv + nc, generator=gen, device="cuda", dtype=torch.float64)
        ev = torch.sort(u[:nv] * 10.0 - 10.0)[0] * EV
        ec = torch.sort((5.0 ** 1.5 + u[nv:] * (60.0 ** 1.5 - 5.0 ** 1.5)) ** (2.0 / 3.0))[0] * EV
        ncol = col = None
        if nw:   # the last columns are windows: representatives of 30 eV and up with their counts
            k = torch.arange(nw, device="cuda", dtype=torch.float64)
            ec[nc - nw:] = (30.0 + (k + 0.5) * 30.0 / nw) * EV
            ncol = torch.ones(nc, device="cuda", dtype=torch.float64)
            ncol[nc - nw:] = torch.round(300.0 + 500.0 * torch.rand(nw, generator=gen, device="cuda",
                                                                    dtype=torch.float64))
            col = torch.arange(nc, device="cuda", dtype=torch.int32)
        probs.append((cv.contiguous(), ev.contiguous(), cc.contiguous(), ec.contiguous(), ncol, col))
    return probs


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _response(gen, ng, nb, a, hermitian):
    """chi0-like matrices: a correlation matrix between rows that fall off with |q+G|, negative
    semidefinite; a dynamic one has a smaller anti-Hermitian part."""
    g = _chi_sphere(ng, QS[0])
    k2 = (((g + np.array(QS[0])) * (2.0 * math.pi / a)) ** 2).sum(1)
    d = torch.from_numpy(np.sqrt(k2) / (1.0 + k2)).cuda() * math.sqrt(a ** 3 * 0.2)
    out = []
    for _ in range(nb):
        b = torch.randn((ng, 64), generator=gen, device="cuda", dtype=C128) * 0.1
        m = b @ b.conj().T + torch.eye(ng, device="cuda", dtype=C128)
        if not hermitian:
            b = torch.randn((ng, 64), generator=gen, device="cuda", dtype=C128) * 0.05
            m = 0.7 * m + 0.3j * (b @ b.conj().T + torch.eye(ng, device="cuda", dtype=C128))
        out.append(-(d[:, None] * m * d[None, :]))
    v = torch.from_numpy(_coulomb(a, g, QS[0])).cuda()
    return v, torch.stack(out)


def _modes(gen, ng, a):
    """Omega^2 and wt^2 of a plasmon-pole model: poles of 10 to 30 eV, off-diagonal ones complex."""
    o = torch.randn((ng, ng), generator=gen, device="cuda", dtype=C128)
    w = (10.0 + 20.0 * torch.rand((ng, ng), generator=gen, device="cuda", dtype=torch.float64)) * EV
    wt2 = (w * w) * torch.exp(0.3j * torch.randn((ng, ng), generator=gen, device="cuda", dtype=torch.float64))
    wp2 = 4.0 * math.pi * 256.0 / a ** 3 / 16.0
    fall = torch.exp(-0.003 * torch.arange(ng, device="cuda", dtype=torch.float64))
    om2 = wp2 * (0.05 * o * fall[:, None] * fall[None, :] + torch.eye(ng, device="cuda", dtype=C128))
    return torch.stack([om2, wt2])


def _inputs(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind == "inverse":
        return _response(gen, case["ng"], case["nbatch"], 16.8, case["hermitian"])
    nd = case["nd"]
    a = _lattice(nd)
    probs = _bands(case, gen, len(_wf_sphere(nd)))
    if kind == "adjoint":
        ng = case["ng"]
        x = torch.randn((case["nomega"], ng, ng), generator=gen, device="cuda", dtype=C128)
        return probs, x
    if kind in ("coh", "gpp"):
        v = torch.from_numpy(_coulomb(a, _chi_sphere(case["ng"], QS[0]), QS[0])).cuda()
        v[0] = v[1:].max()   # the head is averaged over the cell around q = 0
        if kind == "gpp":
            return probs, v, _modes(gen, case["ng"], a)
        b = torch.randn((case["ng"], 32), generator=gen, device="cuda", dtype=C128) * 0.05
        return probs, v, torch.eye(case["ng"], device="cuda", dtype=C128) * 0.5 + b @ b.conj().T * 0.1
    return probs


def _energies(case):
    return [(-8.0 + 3.0 * j) * EV for j in range(case["nenergy"])]


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": dict(case), "own": _Geometry()}
    ctx = st["own"].ctx
    data = _inputs(case, seed)
    if kind == "inverse":
        st["v"], st["chi"] = data
        st["ws"] = torch.empty(gw.gw_eps_inv_workspace_size(ctx, case["ng"], case["nbatch"]), dtype=torch.uint8,
                               device="cuda")
        return st
    nd = case["nd"]
    probs = data if kind == "build" else data[0]
    recs = []
    for iq, (n, p) in enumerate(zip(_ngs(case), probs)):
        geom = st["own"].add(nd, _wf_sphere(nd), _chi_sphere(n, QS[iq]), _lattice(nd), QS[iq])
        cv, ev, cc, ec, ncol, col = p
        recs.append(gw.make_problem(geom, cv, ev, cc, ec, ncol, col))
    st["probs"] = recs
    if kind in ("build", "adjoint"):
        st["prec"] = gw.PRECISIONS[case["prec"]]
        n = gw.gw_chi0_workspace_size(ctx, recs, case["nomega"], st["prec"])
    elif kind == "coh":
        n = gw.gw_sigma_coh_workspace_size(ctx, recs[0])
    else:
        n = 0
    st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    if kind != "build":
        st["more"] = data[1:]
    return st


def run(st):
    case = st["case"]
    kind, ctx = case["kind"], st["own"].ctx
    if kind == "inverse":
        return gw.gw_eps_inv(ctx, st["v"], st["chi"], workspace=st["ws"], hermitian=case["hermitian"])
    if kind == "coh":
        return gw.gw_sigma_coh_static(ctx, st["probs"][0], st["more"][0], st["more"][1], workspace=st["ws"])
    if kind == "gpp":
        return gw.gw_sigma_coh_gpp(ctx, st["probs"], [st["more"][0]], [st["more"][1]], _energies(case), 0.1 * EV)
    om, delta = _omegas(case)
    if kind == "build":
        chi = gw.gw_chi0_build(ctx, st["probs"], _ngs(case), om, delta, st["prec"], workspace=st["ws"])
        # the mixed precisions carry about seven digits: their matrices are kept in single precision
        return chi if case["prec"] == "fp64" else [x.to(torch.complex64) for x in chi]
    g = gw.gw_chi0_backward(ctx, st["probs"], om, delta, st["prec"], st["more"][0], workspace=st["ws"],
                            coef=(case["coef"], case["coef"]))
    return list(g) if case["prec"] == "fp64" else [x.float() for x in g]


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "inverse":
        n, b = float(case["ng"]), case["nbatch"]
        return {"bytes": b * 32.0 * n * n, "flops": b * (4.0 if case["hermitian"] else 8.0) * n ** 3}
    nd, nv, nc = case["nd"], case["nv"], case["ncol"]
    npw = len(_wf_sphere(nd))
    flops = bts = 0.0
    for n, iq in zip(_ngs(case), range(4)):
        rc = int(np.abs(_chi_sphere(n, QS[iq])).max())
        nn = 2 * (nd // 4) + rc + 1      # the smallest grid that holds the product without aliasing
        k, lg = 2 * rc + 1, math.log2(nn)
        pair = 5.0 * nn ** 3 * lg * (1.0 + k / nn + (k / nn) ** 2) + 6.0 * nn ** 3
        band = 15.0 * nn ** 3 * lg
        flops += pair * nv * nc + band * (nv + nc)
        bts += 16.0 * npw * (nv + nc)
        nw = case.get("nomega", 1)
        if kind == "build":
            flops += (4.0 if nw == 1 else 8.0 * nw) * n * n * nv * nc
            bts += 16.0 * nw * n * n
        elif kind == "adjoint":
            flops += 8.0 * nw * n * n * nv * nc
            bts += 16.0 * nw * n * n
            if case["coef"]:
                flops += 16.0 * nw * n * n * nv * nc + pair * nv * nc + band * (nv + nc) + 16.0 * nn ** 3 * nv * nc
                bts += 16.0 * npw * (nv + nc)
        elif kind == "coh":
            flops += 8.0 * n * n * nv * nc
            bts += 16.0 * n * n
        else:
            flops += n * n * nc * case["nenergy"] * (12.0 + 8.0 * nv)
            bts += 32.0 * n * n
    return {"bytes": bts, "flops": flops}


# ---------------------------------------------------------------- the same in plain torch, 64 bits
def _fft_size(n):
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


class _Transform:
    """Band rows on the grid, and the pair densities of a block of columns."""

    def __init__(self, nd, ng, iq):
        wf, chi = _wf_sphere(nd).astype(np.int64), _chi_sphere(ng, QS[iq]).astype(np.int64)
        n = self.n = _fft_size(2 * int(np.abs(wf).max()) + int(np.abs(chi).max()) + 1)
        flat = lambda g: torch.from_numpy(((g[:, 0] % n) * n + g[:, 1] % n) * n + g[:, 2] % n).cuda()  # noqa: E731
        self.wf, self.chi = flat(wf), flat(chi)

    def real(self, coef):
        n = self.n
        box = torch.zeros((coef.shape[0], n ** 3), dtype=C128, device="cuda")
        box[:, self.wf] = coef
        return torch.fft.ifftn(box.view(-1, n, n, n), dim=(1, 2, 3), norm="forward")

    def pairs(self, uv, uc):
        """(nv * nc, ng) of conj(uv) uc, a few hundred pairs at a time."""
        n, out = self.n, []
        step = max(1, int(3e9 / 16 / n ** 3))
        for v in range(uv.shape[0]):
            rows = [torch.fft.ifftn(uv[v].conj()[None] * uc[c:c + step], dim=(1, 2, 3)).view(-1, n ** 3)[:, self.chi]
                    for c in range(0, uc.shape[0], step)]
            out.append(torch.cat(rows))
        return torch.stack(out)


def _weights(ev, ec, ncol, om, delta, deriv=False):
    """Weights w (nv, nc) of Eq. (chi0), and dw/dx for x = E_v - E_c."""
    x = (ev[:, None] - ec[None, :]).to(C128)
    n = 1.0 if ncol is None else ncol[None, :]
    a, b = 1.0 / (x - om + 1j * delta), 1.0 / (x + om + 1j * delta)
    w = 0.5 * n * (a + b)
    return (w, -0.5 * n * (a * a + b * b)) if deriv else w


def _blocks(case, ng, nc):
    step = max(1, int(6e9 / 16 / ng / case["nv"]))
    return [(c, min(nc, c + step)) for c in range(0, nc, step)]


def exact(case, seed):
    if _seconds(case) > 2.0:
        return None
    kind = case["kind"]
    data = _inputs(case, seed)
    if kind == "inverse":
        v, chi = data
        eye = torch.eye(case["ng"], device="cuda", dtype=C128)
        return torch.stack([torch.linalg.inv(eye - v[:, None] * x) for x in chi])
    om, delta = _omegas(case)
    probs = data if kind == "build" else data[0]
    if kind == "build":
        res = []
        for iq, (ng, (cv, ev, cc, ec, ncol, col)) in enumerate(zip(_ngs(case), probs)):
            t = _Transform(case["nd"], ng, iq)
            uv = t.real(cv)
            chi = torch.zeros((len(om), ng, ng), dtype=C128, device="cuda")
            for c0, c1 in _blocks(case, ng, len(ec)):
                m = t.pairs(uv, t.real(cc[c0:c1])).view(-1, ng)
                for i, w in enumerate(om):
                    wt = _weights(ev, ec[c0:c1], None if ncol is None else ncol[c0:c1], w, delta).reshape(-1, 1)
                    chi[i] += (wt * m).T @ m.conj()
                del m
            res.append(chi if case["prec"] == "fp64" else chi.to(torch.complex128))
        return res
    cv, ev, cc, ec, ncol, col = probs[0]
    ng, nv, nc = case["ng"], case["nv"], case["ncol"]
    t = _Transform(case["nd"], ng, 0)
    uv = t.real(cv)
    if kind == "adjoint":
        return _exact_adjoint(case, t, uv, probs[0], data[1], om, delta)
    v, x = data[1], data[2]
    blocks = _blocks(case, ng, nc)
    if kind == "coh":
        s = torch.zeros((nv, nv), dtype=C128, device="cuda")
        kern = (x - torch.eye(ng, device="cuda", dtype=C128)) * v[None, :]
        for c0, c1 in blocks:
            m = t.pairs(uv, t.real(cc[c0:c1]))
            if ncol is not None:
                left = m * ncol[None, c0:c1, None]
            else:
                left = m
            z = (left.reshape(-1, ng) @ kern).view(nv, -1)
            s += 0.5 * z @ m.reshape(nv, -1).conj().T
        return s
    en = _energies(case)
    s = torch.zeros((len(en), nv, nv), dtype=C128, device="cuda")
    wt = torch.sqrt(x[1])
    b = x[0] * v[None, :] / wt
    for c0, c1 in blocks:
        m = t.pairs(uv, t.real(cc[c0:c1]))
        for c in range(c0, c1):
            mc, e = m[:, c - c0].contiguous(), float(ec[c])
            wc = 1.0 if ncol is None else float(ncol[c])
            for j, ej in enumerate(en):
                s[j] += 0.5 * wc * (mc @ (b / (ej - e + 0.1j * EV - wt))) @ mc.conj().T
    return s


def _exact_adjoint(case, t, uv, prob, x, om, delta):
    cv, ev, cc, ec, ncol, col = prob
    ng, n = case["ng"], t.n
    gv = torch.zeros_like(ev)
    gc, gn = torch.zeros_like(ec), torch.zeros_like(ec)
    gcv = torch.zeros_like(uv) if case["coef"] else None
    gcc = []
    for c0, c1 in _blocks(case, ng, len(ec)):
        uc = t.real(cc[c0:c1])
        m = t.pairs(uv, uc)
        flat = m.view(-1, ng)
        mbar = torch.zeros_like(flat)
        nw = None if ncol is None else ncol[c0:c1]
        for i, w in enumerate(om):
            y = flat @ x[i].T
            s = (flat.conj() * y).sum(1).view(len(ev), -1)
            wt, dw = _weights(ev, ec[c0:c1], nw, w, delta, deriv=True)
            dx = (s.conj() * dw).real
            gv += dx.sum(1)
            gc[c0:c1] -= dx.sum(0)
            gn[c0:c1] += (s.conj() * _weights(ev, ec[c0:c1], None, w, delta)).real.sum(0)
            if case["coef"]:
                mbar += wt.conj().reshape(-1, 1) * y + wt.reshape(-1, 1) * (flat @ x[i].conj())
        if case["coef"]:
            mbar = mbar.view(len(ev), c1 - c0, ng)
            ubar = torch.zeros_like(uc)
            for v in range(len(ev)):
                for b0 in range(0, c1 - c0, 64):
                    sl = slice(b0, min(c1 - c0, b0 + 64))
                    box = torch.zeros((sl.stop - b0, n ** 3), dtype=C128, device="cuda")
                    box[:, t.chi] = mbar[v, sl]
                    h = torch.fft.fftn(box.view(-1, n, n, n), dim=(1, 2, 3)) / n ** 3
                    ubar[sl] += h * uv[v][None]
                    gcv[v] += (h.conj() * uc[sl]).sum(0)
            gcc.append(torch.fft.fftn(ubar, dim=(1, 2, 3)).view(-1, n ** 3)[:, t.wf])
    out = [gv, gc, gn]
    if case["coef"]:
        out += [torch.fft.fftn(gcv, dim=(1, 2, 3)).view(-1, n ** 3)[:, t.wf].reshape(-1), torch.cat(gcc).reshape(-1)]
    return out
