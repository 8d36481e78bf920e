"""The float64 pair planes on both sides of each change of shape: up to max|n_chi| = 7 at 64 and 68 points; 8 and 9
at 76 and 80, with fewer row quads than a step holds, a last step of one, two and three of them; 12, 13 and 15 at
the largest grid of the two-quad shape and beyond it; and the largest float64 grid, 104.  Against the oracle on the
stated grid.

Tolerance 1e-10, as for the other float64 parity tests."""
import numpy as np
import pytest

import oracle
from test_gpu_folded import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd,rw,rc,nt", [
    (64, 28, 7, 64), (72, 29, 7, 68), (72, 31, 2, 68), (104, 48, 7, 104), (88, 40, 4, 88),
    (24, 4, 8, 20), (24, 5, 9, 20), (24, 7, 9, 24), (32, 9, 8, 28), (72, 31, 9, 72), (80, 33, 9, 76), (80, 33, 8, 76),
    (80, 34, 9, 80), (80, 35, 8, 80), (104, 47, 9, 104), (96, 41, 9, 92),
    (104, 45, 12, 104), (96, 41, 13, 96), (104, 43, 13, 100), (88, 36, 15, 88), (96, 38, 15, 92)])
def test_float64_planes_on_both_sides_of_each_shape(gpu, nd, rw, rc, nt):
    import torch
    import paper_1601_06767_amd as p
    assert nt == min(nd, -(-max(2 * rw + rc + 1, 2 * rc + 1, 16) // 4) * 4)   # points of the transforms
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, 5, 9, nt % 8 == 4)
    ref = oracle.chi0_bands(cv, ev, cc, ec, gw, gc, (nd,) * 3)[0]
    dev = torch.device("cuda", 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        prob = p.make_problem(geom, *ts)
        for _ in range(2):   # the second pass finds the first one's values in the scratch memory
            chi = p.gw_chi0_build(ctx, [prob], [len(gc)], [0.0], 0.0, p.GW_FP64)[0][0].cpu().numpy()
            err = np.linalg.norm(chi - ref) / np.linalg.norm(ref)
            print(f"N {nd}, rw {rw}, rc {rc}: {err:.2e}", flush=True)
            assert err <= 1e-10 and np.abs(chi - ref).max() <= 1e-10 * np.abs(ref).max(), err
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)
