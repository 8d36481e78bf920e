"""Column counts that are odd multiples of eight, in one chunk and in several: the columns of a call are
padded to eight, no further, and a chunk's length may be an odd number of eights (twelve valence bands:
2728 columns).  chi0 is a sum over columns, so the call must equal the sum of two calls that share them:
to 1e-12 in float64 (sums of 32k terms in another order), 1e-6 and 1e-5 in float32 and split-bf16 (of the
norm; the float32 sums of a range and the split of a factor, as in the other parity tests)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup(gpu):
    import torch
    import paper_1601_06767_amd as p
    q = (0.01, 0.0, 0.0)
    gw, gc = synth.wf_sphere(8, 4), synth.chi_sphere(130, q, np.eye(3) * 8.0)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (24,) * 3, gw, gc)
    r = np.random.default_rng(8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    coef = lambda n: (r.standard_normal((n, len(gw))) + 1j * r.standard_normal((n, len(gw)))) / np.sqrt(2 * len(gw))
    yield p, ctx, geom, t, coef, r, len(gc)
    p.gw_geom_destroy(geom)
    p.gw_ctx_destroy(ctx)


def test_columns_are_padded_to_eight(setup):
    p, ctx, geom, t, coef, r, ng = setup
    for nv in (4, 200, 3000):
        ev, cv = t(r.uniform(-0.4, 0.0, nv)), t(coef(nv))
        ws = {}
        for nc in (8, 16, 40, 48):
            prob = p.make_problem(geom, cv, ev, t(coef(nc)), t(r.uniform(0.2, 2.0, nc)))
            for prec in (p.GW_FP64, p.GW_FP32, p.GW_BF16X3):
                ws[nc, prec] = p.gw_chi0_workspace_size(ctx, [prob], 1, prec)
        for prec in (p.GW_FP64, p.GW_FP32, p.GW_BF16X3):
            if nv < 3000:
                assert ws[8, prec] < ws[16, prec] and ws[40, prec] < ws[48, prec]
            else:   # a chunk holds eight columns, however many there are
                assert ws[8, prec] == ws[48, prec]


def test_band_scratch_is_for_the_bands_of_the_call(setup):
    # eight columns beside four valence bands: everything of theirs, the transforms' scratch included, is a
    # fifth of what forty columns take
    p, ctx, geom, t, coef, r, ng = setup
    size = {}
    for nc in (8, 40):
        prob = p.make_problem(geom, t(coef(4)), t(np.zeros(4)), t(coef(nc)), t(np.ones(nc)))
        size[nc] = p.gw_chi0_workspace_size(ctx, [prob], 1, p.GW_FP64)
    assert 2 * size[8] < size[40], size


@pytest.mark.parametrize("nv,nc,cut", [(5, 8, 3), (5, 40, 17), (12, 2735, 1000), (12, 5460, 2728), (20, 1640, 1632)])
def test_call_equals_sum_of_its_parts(setup, nv, nc, cut):
    import torch
    p, ctx, geom, t, coef, r, ng = setup
    cv, ev, cc, ec = t(coef(nv)), t(r.uniform(-0.4, 0.0, nv)), t(coef(nc)), t(r.uniform(0.2, 2.0, nc))
    prob = lambda a, b: p.make_problem(geom, cv, ev, cc[a:b], ec[a:b])
    for prec, tol in ((p.GW_FP64, 1e-12), (p.GW_FP32, 1e-6), (p.GW_BF16X3, 1e-5)):
        whole, one, two = (p.gw_chi0_build(ctx, [x], [ng], [0.0], 0.0, prec)[0].clone()
                           for x in (prob(0, nc), prob(0, cut), prob(cut, nc)))
        err = float((whole - one - two).norm() / whole.norm())
        print(f"{nv} x {nc}: {err:.1e}", flush=True)
        assert err <= tol
