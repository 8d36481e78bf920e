"""The rounding of the pair densities in the split-bf16 adjoint without broadening, alone: chibar of small
integers, which one bf16 part holds exactly (and so the sums chibar + chibar^H), leaves only the split of M,
whose parts hi + lo + residual hold all 24 bits of a float32, and float32 sums of up to 259 products.

Tolerance 1e-6, rms over the columns relative to their rms: float32 pair densities (1.8e-7 of the norm, which
enter twice) and float32 sums (2^-24 a term, a few hundred terms: 4e-7); without the residual the split alone
makes 2e-6 (2^-18 / sqrt 3 of each value, counted twice)."""
import numpy as np
import pytest

from cases import make_case
from test_gpu_adjoint import g, gpu_backward, ref_backward  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hermitian", [False, True])
def test_pair_densities_enter_with_all_their_bits(g, hermitian):
    case = make_case(0, nv=8, nc=64)
    ng = len(case.gc)
    r = np.random.default_rng(2)
    gbar = (r.integers(-8, 9, (1, ng, ng)) + 1j * r.integers(-8, 9, (1, ng, ng))).astype(complex)
    if hermitian:
        gbar = gbar + gbar.conj().transpose(0, 2, 1)
    got, want = gpu_backward(g, case, gbar, [0.0], 0.0, "bf16x3"), ref_backward(case, gbar, [0.0], 0.0)
    for name, a, b in zip(("e_v", "e_col", "n_col"), got, want):
        err = float(np.sqrt(np.mean((np.asarray(a) - b) ** 2) / np.mean(b ** 2)))
        print(f"{name}: {err:.2e}", flush=True)
        assert err <= 1e-6, (name, err)
