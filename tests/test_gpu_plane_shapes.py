"""The float32 pair planes at chunkings the other shape tests leave out: transform grids of 52 to 112
points (chunks of x3 quads in fours and sixes, an empty last chunk, short last chunks and row steps), on
both sides of the change of shape between max|n_chi| = 7 and 8.  Against the oracle on the stated grid.

Tolerance 2e-5, as for the other float32 parity tests (pair densities of relative error ~1e-7, float32
sums of up to some hundred pairs); float64 1e-10."""
import numpy as np
import pytest

import oracle
from test_gpu_folded import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd,rw,rc", [(104, 46, 7), (112, 51, 8), (88, 36, 9), (56, 22, 7), (88, 40, 6)])
def test_plane_chunks_match_oracle(gpu, nd, rw, rc):
    import torch
    import paper_1601_06767_amd as p
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, 3, 9, False)
    ref = oracle.chi0_bands(cv, ev, cc, ec, gw, gc, (nd,) * 3)[0]
    dev = torch.device("cuda", 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        prob = p.make_problem(geom, *ts)
        for _ in range(2):   # the second pass finds the first one's values in the scratch memory
            chi = p.gw_chi0_build(ctx, [prob], [len(gc)], [0.0], 0.0, p.GW_FP32)[0][0].cpu().numpy()
            err = np.linalg.norm(chi - ref) / np.linalg.norm(ref)
            print(f"N {nd}, rw {rw}, rc {rc}: {err:.2e}", flush=True)
            assert err <= 2e-5 and np.abs(chi - ref).max() <= 2e-5 * np.abs(ref).max(), err
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)


@pytest.mark.parametrize("nd,rw,rc", [(88, 36, 5), (104, 46, 3), (104, 48, 3)])
def test_band_slabs_of_every_lds_form_match_oracle(gpu, nd, rw, rc):
    # float64 slabs with the factors, but not the coefficients, beside them in LDS, and with neither
    import torch
    import paper_1601_06767_amd as p
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, 2, 3, False)
    ref = oracle.chi0_bands(cv, ev, cc, ec, gw, gc, (nd,) * 3)[0]
    dev = torch.device("cuda", 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        chi = p.gw_chi0_build(ctx, [p.make_problem(geom, *ts)], [len(gc)], [0.0], 0.0, p.GW_FP64)[0][0].cpu().numpy()
        err = np.linalg.norm(chi - ref) / np.linalg.norm(ref)
        print(f"N {nd}, rw {rw}, rc {rc}: {err:.2e}", flush=True)
        assert err <= 1e-10 and np.abs(chi - ref).max() <= 1e-10 * np.abs(ref).max(), err
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)


@pytest.mark.parametrize("nd,rw,rc", [(32, 14, 3), (40, 14, 4), (32, 13, 5), (16, 3, 1)])
def test_float64_planes_on_both_sides_of_the_small_shape(gpu, nd, rw, rc):
    # 32 points and 36, max|n_chi| 4 and 5; several workgroups of pairs
    import torch
    import paper_1601_06767_amd as p
    gw, gc, cv, ev, cc, ec = _case(nd, rw, rc, 6, 21, False)
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
