"""Pair densities whose rows in the sphere's order fit the LDS of the x1 stage exactly, or not any more:
10,240 values of 16 bytes and one more, in float32 20,480 of 8 bytes and one more, and a row that is mostly
padding.  Against the product on the stated grid.

Tolerance: three axes of at most 32 additions each, half a unit in the last place per addition: 96 x 2^-24 =
5.7e-6 in float32 and 1.1e-14 in float64, relative to the sums' terms; twice that of the norm, with the
same again for the bands' transform."""
import numpy as np
import pytest

import oracle
from test_gpu_folded import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rc,ng,prec", [(11, 10240, "fp64"), (11, 10241, "fp64"), (11, 12167, "fp64"),
                                        (14, 20480, "fp32"), (14, 20481, "fp32"), (11, 130, "fp32"), (1, 27, "fp64")])
def test_rows_on_both_sides_of_the_lds_size(gpu, rc, ng, prec):
    import torch
    import paper_1601_06767_amd as p
    nd, rw, nv, nc = 32, 3, 4, 8
    gw, _, cv, ev, cc, ec = _case(nd, rw, 1, nv, nc, False)
    a = np.arange(-rc, rc + 1)
    gc = np.stack(np.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    gc = np.ascontiguousarray(np.random.default_rng(rc).permutation(gc)[:ng].astype(np.int32))
    ref = oracle.pair_density_fft(oracle.psi_real_space(cv, gw, (nd,) * 3), oracle.psi_real_space(cc, gw, (nd,) * 3), gc)
    dev = torch.device("cuda", 0)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc)
    try:
        ts = [t(cv), t(ev), t(cc), t(ec)]
        prob = p.make_problem(geom, *ts)
        for _ in range(2):   # the second pass finds the first one's values in the scratch memory
            m = p.gw_pair_density(ctx, prob, 0, nv, 0, nc, ng, p.PRECISIONS[prec]).cpu().numpy()
            err = np.linalg.norm(m - ref) / np.linalg.norm(ref)
            print(f"rc {rc}, {ng} G, {prec}: {err:.2e}", flush=True)
            assert err <= 4 * 96 * (2.0 ** -24 if prec == "fp32" else 2.0 ** -53), err
    finally:
        p.gw_geom_destroy(geom)
        p.gw_ctx_destroy(ctx)
