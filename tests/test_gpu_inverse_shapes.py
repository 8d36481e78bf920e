"""The dielectric inverse at the edges of its launch shapes: row counts around what a workgroup of
the pivot steps holds (multiples of 512 up to 2048) and beyond it, partial panels and sub-panels,
batches with a workspace for one matrix and for several, and matrices whose every pivot is off the
diagonal.  Tolerance: 1e-11 of the largest entry, as the other inverse tests (float64, condition
numbers of a few hundred at most)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _chi(n, herm, seed):
    r = np.random.default_rng(seed)
    a = (r.standard_normal((n, n)) + 1j * r.standard_normal((n, n))) / np.sqrt(n)
    return -(a @ a.conj().T) / 4.0 if herm else a / 3.0


@pytest.fixture
def ctx(gpu):
    import paper_1601_06767_amd as p
    c = p.gw_ctx_create(0)
    yield c
    p.gw_ctx_destroy(c)


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n", [1, 2, 15, 17, 63, 65, 129, 512, 513, 1024, 1025, 1537, 2048, 2049, 2113])
def test_inverse_matches_lapack_at_shape_edges(ctx, n):
    import paper_1601_06767_amd as p
    v = np.random.default_rng(n).uniform(0.5, 2.0, n)
    for herm in (False, True):
        chi = _chi(n, herm, 7 * n + herm)
        z = p.gw_eps_inv(ctx, _t(v), _t(chi), hermitian=herm)
        p.gw_eps_inv_status(ctx)
        ref = oracle.eps_inv(chi, v)
        err = float(np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max())
        print(f"n = {n}, hermitian = {herm}: {err:.1e}", flush=True)
        assert err <= 1e-11


@pytest.mark.parametrize("n", [70, 600, 1100, 2060])
def test_pivots_off_the_diagonal(ctx, n):
    # eps = a cyclic shift by a third of the rows plus a small matrix: every pivot is a row interchange
    import paper_1601_06767_amd as p
    r = np.random.default_rng(n)
    eps = np.roll(np.eye(n), n // 3, axis=0) + 1e-3 * (r.standard_normal((n, n)) + 1j * r.standard_normal((n, n)))
    np.fill_diagonal(eps, 0.0)
    v = np.ones(n)
    chi = np.eye(n) - eps
    z = p.gw_eps_inv(ctx, _t(v), _t(chi), hermitian=False)
    p.gw_eps_inv_status(ctx)
    ref = np.linalg.inv(eps)
    assert np.abs(z.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("herm", [False, True])
def test_batches_do_not_depend_on_the_workspace(ctx, herm):
    import torch
    import paper_1601_06767_amd as p
    n, nb = 333, 5
    chi = np.stack([_chi(n, herm, 50 + b) for b in range(nb)])
    v = np.random.default_rng(5).uniform(0.5, 2.0, (nb, n))
    one = p.gw_eps_inv_workspace_size(ctx, n, 1)
    full = p.gw_eps_inv_workspace_size(ctx, n, nb)
    assert full >= 2 * one
    got = [p.gw_eps_inv(ctx, _t(v), _t(chi), workspace=torch.empty(b, dtype=torch.uint8, device="cuda:0"), hermitian=herm)
           for b in (one, 2 * one + 100, full)]
    p.gw_eps_inv_status(ctx)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    for b in range(nb):
        ref = oracle.eps_inv(chi[b], v[b])
        assert np.abs(got[2][b].cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()
    # a singular matrix anywhere in the batch is reported
    bad = chi.copy()
    v[3] = 1.0
    bad[3] = np.eye(n)   # I - v chi0 = 0 exactly
    p.gw_eps_inv(ctx, _t(v), _t(bad), hermitian=herm)
    with pytest.raises(p.GwError) as e:
        p.gw_eps_inv_status(ctx)
    assert e.value.status == p.GW_ESINGULAR
