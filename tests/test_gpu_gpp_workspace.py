"""The workspace of the plasmon-pole COH sum over its range of spheres, states and energies, and a sum whose
last chunk of columns is cut into fewer shares than the first.

Bound: eight energies of one pair of state blocks take the partial sums of at most two full sets per 64 x 64
tile (four sums of eight energies and 64 state pairs each, 32 KiB), or 16 MiB where that is more.  Tolerance
of the sum: 1e-10 of the largest element, as for the other float64 parity tests of this sum."""
import ctypes
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from test_gpu_sigma import g, gpp_modes, rel, run_gpp, screened  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _workspace(p, ctx, prob, nenergy):
    n = ctypes.c_size_t()
    arr = p._lib._probs([prob])
    p._lib._check(p._lib.lib.gw_sigma_coh_gpp_workspace_size(ctx, arr, 1, nenergy, ctypes.byref(n)), ctx)
    return n.value


@pytest.mark.parametrize("ng", [64, 259, 800, 1114, 1429, 2000, 2500, 4000, 6000, 8000])
def test_partial_sums_stay_bounded(g, ng):
    p = g.p
    q = (0.01, 0.0, 0.0)
    geom = p.gw_geom_create(g.ctx, (128,) * 3, synth.wf_sphere(8, 2), synth.chi_sphere(ng, q, np.eye(3) * 20.0))
    try:
        tiles = (-(-ng // 128) * 2) ** 2
        for states, ncol in ((1, 3), (8, 300), (16, 300), (32, 5000)):
            z = np.zeros
            prob = p.make_problem(geom, g.t(z((states, 1), complex)), g.t(z(states)), g.t(z((ncol, 1), complex)),
                                  g.t(z(ncol)))
            blocks = (-(-states // 8)) ** 2
            eight = _workspace(p, g.ctx, prob, 16) - _workspace(p, g.ctx, prob, 8)
            print(f"NG {ng}, {states} states: {eight / 2**20:.1f} MiB per eight energies", flush=True)
            assert eight <= blocks * max(2 * tiles * 32 * 1024, 16 << 20), (states, eight)
    finally:
        p.gw_geom_destroy(geom)


def test_short_last_chunk_of_columns(g, screened, gpp_modes):
    # 8 states make a chunk of 4096 columns: 16 shares on the four tiles of this sphere, then three columns
    case, _, v = screened
    _, om2, wt2 = gpp_modes
    ng = 64
    small = dataclasses.replace(case, gc=case.gc[:ng])
    om2, wt2, v = om2[:ng, :ng].copy(), wt2[:ng, :ng].copy(), v[:ng]
    r = np.random.default_rng(4)
    states = np.concatenate([case.coef_v, case.coef_c])[-8:]
    col = r.integers(0, len(case.coef_c), 4099)
    e_col, w = np.sort(r.uniform(0.2, 2.0, len(col))), r.uniform(0.5, 2.0, len(col))
    energies = [-0.2, 0.1]
    probs, vs, ms = run_gpp(g, [(small, states, case.coef_c, e_col, w, col, v, om2, wt2)])
    got = g.p.gw_sigma_coh_gpp(g.ctx, probs, vs, ms, energies, 0.003).cpu().numpy()
    # the oracle's sum, with the pair densities of the 240 bands formed once
    nd = (case.nd,) * 3
    m = oracle.pair_density_fft(oracle.psi_real_space(states, case.gw, nd), oracle.psi_real_space(case.coef_c, case.gw, nd),
                                small.gc)
    want = np.zeros_like(got)
    for j, e in enumerate(energies):
        for c, b in enumerate(col):
            a = oracle.gpp_coh_kernel(om2, wt2, v, e - e_col[c] + 0.003j)
            want[j] += 0.5 * w[c] * (m[:, b] @ a @ m[:, b].conj().T)
    assert rel(got, want) <= 1e-10, rel(got, want)
