"""The folded line transforms and their grid choice at the edges of their ranges: dielectric
spheres of every class of group counts, transform grids of 16 points up to the stated grid, with an
odd and an even number of quads, on both sides of each shape's largest grid, spheres that are not
balls, and column counts that are not whole workgroups.  Against the oracle on the stated grid.

Tolerances: float64 1e-10; float32 2e-5 and split-bf16 1e-4 (the bounds of the other parity tests:
float32 pair densities of relative error ~1e-7, float32 sums of up to some thousand pairs)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _ball(r):
    return synth.wf_sphere(8, r)


def _case(nd, rw, rc, nv, nc, odd):
    gw = _ball(rw)
    gc = _ball(rc)
    if odd:   # a lopsided set: no inversion symmetry, empty lines at one side
        gc = gc[(gc[:, 1] >= -1) & ((gc[:, 2] + 2 * gc[:, 0]) % 3 != 1) | (np.abs(gc).max(1) == rc)]
    r = np.random.default_rng(nd * 1000 + rw * 10 + rc)
    coef = lambda n: (r.standard_normal((n, len(gw))) + 1j * r.standard_normal((n, len(gw)))) / np.sqrt(2 * len(gw))
    return gw, np.ascontiguousarray(gc), coef(nv), np.sort(r.uniform(-0.4, 0.0, nv)), coef(nc), np.sort(
        r.uniform(0.2, 2.0, nc))


SHAPES = [(16, 2, 0, False), (16, 1, 1, False), (16, 4, 3, True), (24, 6, 5, False), (24, 9, 2, True),
          (40, 13, 6, False), (56, 22, 7, False), (56, 23, 7, True), (72, 30, 7, False), (72, 31, 7, False),
          (64, 27, 8, True), (64, 20, 9, False), (48, 14, 10, True), (56, 20, 11, False), (56, 20, 13, False),
          (64, 24, 14, True), (64, 23, 15, False), (128, 56, 15, False)]


@pytest.mark.parametrize("nd,rw,rc,odd", SHAPES, ids=[f"{a}-rw{b}-rc{c}" + ("-odd" if d else "") for a, b, c, d in SHAPES])
def test_folded_transforms_match_oracle(gpu, nd, rw, rc, odd):
    import torch
    import paper_1601_06767_amd as p
    nv, nc = (2, 3) if nd == 128 else (5, 19)
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, nv, nc, odd)
    ref = oracle.chi0_bands(cv, ev, cc, ec, gw, gc, (nd,) * 3)[0]
    dev = torch.device("cuda", 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        prob = p.make_problem(geom, *ts)
        for prec, tol in (("fp64", 1e-10), ("fp32", 2e-5), ("bf16x3", 1e-4)):
            if nd == 128 and prec == "fp64":   # the float64 slab of a band exceeds the LDS: refused
                with pytest.raises(p.GwError):
                    p.gw_chi0_build(ctx, [prob], [len(gc)], [0.0], 0.0, p.GW_FP64)
                continue
            for form in ((0, 1, 2, 3) if prec == "fp32" else (0,)):
                p.gw_tune_set(ctx, prob, p.PRECISIONS[prec], form, 0)
                chi = p.gw_chi0_build(ctx, [prob], [len(gc)], [0.0], 0.0, p.PRECISIONS[prec])[0][0].cpu().numpy()
                err = np.linalg.norm(chi - ref) / np.linalg.norm(ref)
                print(f"N {nd}, rw {rw}, rc {rc}, {prec}, form {form}: {err:.2e}", flush=True)
                assert err <= tol and np.abs(chi - ref).max() <= tol * np.abs(ref).max(), (prec, form, err)
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)
