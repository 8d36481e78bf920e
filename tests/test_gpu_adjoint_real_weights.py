"""The adjoint without broadening, where only the Hermitian part of chibar enters: spheres on both sides of
the 64- and 128-row tiles and the 16-column stages of its kernels, several frequencies, a chibar that is far
from Hermitian, with and without the coefficient gradients (which take another route).  Against the oracle.

Tolerances: 1e-10 (float64) and 1e-5 (float32) of the largest element, as for the other adjoint parity tests:
the same products, each sum over half as many elements of twice the size.  Split-bf16: a factor hi + lo holds
x to 2^-17, uniformly distributed (rms 2^-17 / sqrt 3) in both factors of a product, and a sum of random
products has the same relative error as one product: rms 6.2e-6; the largest of some hundred values stays
under six times that, 3.7e-5."""
import dataclasses

import numpy as np
import pytest

from cases import make_case
from test_gpu_adjoint import close, g, gpu_backward, rand_gbar, ref_backward  # noqa: F401  (fixture)
from test_gpu_coef_grad import err, run, want_coef

pytestmark = pytest.mark.gpu


def _case(ng):
    case = make_case(0, nv=5, nc=13)
    return dataclasses.replace(case, gc=case.gc[:min(ng, len(case.gc))])


@pytest.mark.parametrize("ng", [17, 57, 64, 65, 127, 128, 129, 259])
def test_real_weight_adjoint_tile_edges(g, ng):
    case = _case(ng)
    om = [0.0, 0.01]
    gbar = rand_gbar(len(case.gc), 2, ng)
    want = ref_backward(case, gbar, om, 0.0)
    for prec, tol in (("fp64", 1e-10), ("fp32", 1e-5), ("bf16x3", 3.7e-5)):
        for a, b in zip(gpu_backward(g, case, gbar, om, 0.0, prec), want):
            assert close(a, b, tol), prec


@pytest.mark.parametrize("ng", [57, 65, 259])
def test_real_weight_coefficient_gradients(g, ng):
    case = _case(ng)
    om = [0.0, 0.01]
    gbar = rand_gbar(len(case.gc), 2, ng + 1)
    got = run(g, case, gbar, om, 0.0)
    for a, b in zip(got[:3], ref_backward(case, gbar, om, 0.0)):
        assert close(a, b, 1e-10)
    gv, gc = want_coef(case, gbar, om, 0.0)
    ev, ec = err(got[3].reshape(gv.shape), gv), err(got[4].reshape(gc.shape), gc)
    assert ev <= 1e-10 and ec <= 1e-10, (ev, ec)
