"""Lengths of the pair ranges that the float32 and split-bf16 contractions sum in float32: by themselves
they are cut as finely as the largest split (32), on a small sphere (few tiles) and on one whose rows of M
fill the cache.  A split is a choice of the order of the sums alone, so equal splits give equal bits."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _inputs(rw, ng, nv, nc, seed=0):
    q = (0.01, 0.0, 0.0)
    gw, gc = synth.wf_sphere(8, rw), synth.chi_sphere(ng, q, np.eye(3) * 10.0)
    r = np.random.default_rng(seed)
    coef = lambda n: (r.standard_normal((n, len(gw))) + 1j * r.standard_normal((n, len(gw)))) / np.sqrt(2 * len(gw))
    return gw, gc, coef(nv), np.sort(r.uniform(-0.4, 0.0, nv)), coef(nc), np.sort(r.uniform(0.2, 2.0, nc))


@pytest.mark.parametrize("prec,ng,nv,nc,omegas,delta", [
    ("fp32", 259, 16, 240, [0.0], 0.0), ("fp32", 259, 16, 240, [0.0, 0.3], 0.01), ("bf16x3", 259, 16, 240, [0.0], 0.0),
    ("bf16x3", 259, 16, 240, [0.0, 0.3], 0.01), ("fp32", 4000, 128, 250, [0.0], 0.0)])
def test_float32_ranges_are_cut_as_finely_as_allowed(gpu, prec, ng, nv, nc, omegas, delta):
    import torch
    import paper_1601_06767_amd as p
    gw, gc, cv, ev, cc, ec = _inputs(8, ng, nv, nc)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (32,) * 3, gw, gc)
    try:
        prob = p.make_problem(geom, t(cv), t(ev), t(cc), t(ec))
        build = lambda: p.gw_chi0_build(ctx, [prob], [ng], omegas, delta, p.PRECISIONS[prec])[0]
        own = build()
        p.gw_tune_set(ctx, prob, p.PRECISIONS[prec], 1, 32)
        assert torch.equal(own, build())
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)
