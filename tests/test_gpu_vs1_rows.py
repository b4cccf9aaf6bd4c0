"""One virtual source: every width of the matrix-vector kernels (receiver pairs a lane) at both
ends, with ragged batches, and rejected entries beside a source that is not finite."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, f32, make_plan, random_case, relerr

pytestmark = pytest.mark.gpu

TOL = 1e-5  # float32 sums over up to 4096 receivers and 64 rows


@pytest.mark.parametrize("nb", [1, 3, 13, 64])
@pytest.mark.parametrize("nr", [128, 129, 256, 257, 384, 385, 512, 513, 768, 769, 900, 1024, 1025, 1280, 1281,
                                1664, 1665, 2048, 2049])
def test_every_width(nr, nb):
    ns, nt, nf = 66, 128, 9
    d, u, r = random_case(ns, nr, 1, nt, seed=nr + nb)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = np.random.default_rng(nb).integers(0, ns, size=nb).astype(np.int32)
    it = T(idx, torch.int32)
    assert relerr(H(plan.mdc_forward(T(r), it)), freq.mdc(d[idx], r, nf)) <= TOL
    assert relerr(H(plan.mdc_adjoint(T(u[idx]), it)), freq.mdc_adjoint(d[idx], u[idx], nf)) <= TOL
    G, loss, gn = plan.mdd_stoch_grad(T(r), it)
    lo, go = freq.batch_loss_grad(d, r, u, idx, nf)
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo
    assert abs(gn.item() - np.sum(go ** 2)) <= 2 * TOL * np.sum(go ** 2)


@pytest.mark.parametrize("nr,nb", [(1025, 8), (1025, 9), (1281, 8), (1600, 6), (300, 5)])
def test_many_bins(nr, nb):
    """More frequencies than workgroups that the long rows' registers allow at once."""
    ns, nt, nf = 10, 1024, 513
    d, u, r = random_case(ns, nr, 1, nt, seed=nr)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = np.random.default_rng(nb).integers(0, ns, size=nb).astype(np.int32)
    it = T(idx, torch.int32)
    assert relerr(H(plan.mdc_forward(T(r), it)), freq.mdc(d[idx], r, nf)) <= TOL
    G, loss, _ = plan.mdd_stoch_grad(T(r), it)
    lo, go = freq.batch_loss_grad(d, r, u, idx, nf)
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo


@pytest.mark.parametrize("nb", [3, 20, 40])
@pytest.mark.parametrize("nr", [35, 129, 300, 400, 600, 900, 1100, 1600, 1700, 4000])
def test_rejected_entries_read_no_source(nr, nb):
    """Source 0 is not finite: rejected entries contribute zeros all the same."""
    ns, nt, nf = 50, 128, 9
    d, u, r = random_case(ns, nr, 1, nt, seed=nr + nb)
    d[0] = np.inf
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = np.full(nb, -1, dtype=np.int32)
    G, loss, gn = plan.mdd_stoch_grad(T(r), T(idx, torch.int32))
    assert not H(G).any() and loss.item() == 0.0 and gn.item() == 0.0
    v = f32(np.random.default_rng(nb).standard_normal((nb, 1, nt)))
    assert not H(plan.mdc_adjoint(T(v), T(idx, torch.int32))).any()
    idx[1::2] = np.random.default_rng(nr).integers(1, ns, size=len(idx[1::2]))
    idx[0] = ns
    keep = idx[1::2]
    lo, go = freq.batch_loss_grad(d, r, u, keep, nf)
    G, loss, _ = plan.mdd_stoch_grad(T(r), T(idx, torch.int32))
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo
    assert relerr(H(plan.mdc_adjoint(T(v), T(idx, torch.int32))), freq.mdc_adjoint(d[keep], v[1::2], nf)) <= TOL
    ug = H(plan.mdc_forward(T(r), T(idx, torch.int32)))
    assert relerr(ug[1::2], freq.mdc(d[keep], r, nf)) <= TOL and not ug[0::2].any()
