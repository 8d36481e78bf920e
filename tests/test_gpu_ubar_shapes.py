"""Coefficient gradients at the edges of the shapes of their real-space kernel: grids on both sides of 48 and 64
points (two own bands per workgroup, eight waves of two and of four quads, one and several parts of the
rows), dielectric spheres on both sides of max|n_chi| = 7.  Against the oracle on the stated grid.

Tolerance 1e-10 of the largest element, as for the other float64 gradient parity tests."""
import numpy as np
import pytest

from oracle import grad as og
from test_gpu_folded import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd,rw,rc", [(24, 6, 3), (48, 16, 7), (72, 21, 7), (72, 25, 6), (72, 31, 7), (96, 27, 8),
                                      (96, 30, 9)])
@pytest.mark.parametrize("delta", [0.0, 0.004])
def test_coefficient_gradients_over_plane_shapes(gpu, nd, rw, rc, delta):
    import torch
    import paper_1601_06767_amd as p
    nv, nc = 3, 5
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, nv, nc, False)
    r = np.random.default_rng(nd + rw)
    gbar = (r.standard_normal((1, len(gc), len(gc))) + 1j * r.standard_normal((1, len(gc), len(gc))))
    want = og.grad_chi0_coefficients(cv, ev, cc, ec, gw, gc, (nd,) * 3, gbar, [0.0], delta)
    dev = torch.device("cuda", 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        prob = p.make_problem(geom, *ts)
        got = p.gw_chi0_backward(ctx, [prob], [0.0], delta, p.GW_FP64, t(gbar), coef=(True, True))
        for a, b in zip(got[3:], want):
            a = a.cpu().numpy().reshape(b.shape)
            e = np.abs(a - b).max() / np.abs(b).max()
            print(f"N {nd}, rw {rw}, rc {rc}, delta {delta}: {e:.2e}", flush=True)
            assert e <= 1e-10, e
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)
