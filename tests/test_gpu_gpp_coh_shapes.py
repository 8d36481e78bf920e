"""The plasmon-pole COH sum at the edges of its tiles: one state and one over a block of eight, four and
five energies (one pass and one more), fewer columns than shares and a last share that is short, spheres
of one full 64-tile and one G more, a mode frequency near the largest number.

Tolerance 1e-10 of the largest element, as for the other float64 parity tests of this sum: products and
reciprocals in float64, sums of at most a few thousand terms."""
import dataclasses

import numpy as np
import pytest

import oracle
from test_gpu_sigma import g, gpp_modes, rel, run_gpp, screened  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng,nstates,ncol,nenergy", [(64, 1, 1, 4), (65, 9, 17, 5), (128, 8, 40, 1), (259, 1, 3, 4)])
def test_gpp_coh_tile_edges(g, screened, gpp_modes, ng, nstates, ncol, nenergy):
    case, _, v = screened
    _, om2, wt2 = gpp_modes
    ng = min(ng, len(case.gc))
    small = dataclasses.replace(case, gc=case.gc[:ng])
    om2, wt2, v = om2[:ng, :ng].copy(), wt2[:ng, :ng].copy(), v[:ng]
    wt2[3, 7], om2[3, 7] = 1e308, 1.0   # a mode near the largest number: its term vanishes
    states = np.concatenate([case.coef_v, case.coef_c])[-nstates:]
    cols, e_cols = case.coef_c[:ncol], case.e_c[:ncol]
    energies = list(np.linspace(-0.2, 0.4, nenergy))
    probs, vs, ms = run_gpp(g, [(small, states, cols, e_cols, None, None, v, om2, wt2)])
    got = g.p.gw_sigma_coh_gpp(g.ctx, probs, vs, ms, energies, 0.003).cpu().numpy()
    with np.errstate(over="ignore"):
        want = oracle.sigma_coh_gpp(states, cols, e_cols, case.gw, small.gc, (case.nd,) * 3, om2, wt2, v, energies, 0.003)
    assert np.isfinite(want).all() and got.shape == want.shape
    err = rel(got, want)
    print(f"ng {ng}, {nstates} states, {ncol} columns, {nenergy} energies: {err:.2e}")
    assert err <= 1e-10, err
