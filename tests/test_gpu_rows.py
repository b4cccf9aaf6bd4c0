"""The float32 products at the edges of their tiles: batch rows around multiples of 16,
receivers around the 32-receiver chunks and around the number of chunks that stay in LDS,
columns around the 16-column blocks and the four blocks of a workgroup."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, f32, make_plan, random_case, relerr

pytestmark = pytest.mark.gpu

# The spectra carry float32 rounding of about log2(nt) operations (1e-6 of their norm at
# most) and the compensated products add less than that.
TOL = 2e-6


@pytest.mark.parametrize("prec", ["fp32", "fp32_cgemm"])
@pytest.mark.parametrize("nb,nr,nvs", [(1, 1, 2), (1, 33, 17), (15, 31, 16), (16, 32, 65), (16, 320, 16),
                                       (16, 321, 33), (17, 95, 64), (17, 97, 65), (32, 64, 130),
                                       (33, 63, 18), (48, 65, 66), (49, 129, 20), (64, 40, 81)])
def test_every_kind_at_tile_edges(prec, nb, nr, nvs):
    ns, nt, nf = 70, 128, 41
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb + nr + nvs)
    rng = np.random.default_rng(nb)
    idx = rng.integers(0, ns, size=nb).astype(np.int32)
    if nb > 4:
        idx[1], idx[nb - 1] = -1, ns           # rejected entries act as zero sources
        idx[3] = idx[2]
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision=prec)
    good = (idx >= 0) & (idx < ns)
    keep, ti = idx[good], T(idx, torch.int32)
    out = torch.full((nb, nvs, nt), np.nan, device="cuda")
    ug = H(plan.mdc_forward(T(r), ti, out=out))
    assert relerr(ug[good], freq.mdc(d[keep], r, nf)) <= TOL
    assert not ug[~good].any()
    v = f32(rng.standard_normal((nb, nvs, nt)))
    ga = H(plan.mdc_adjoint(T(v), ti))
    assert relerr(ga, freq.mdc_adjoint(d[keep], v[good], nf)) <= TOL
    G, loss, gn = plan.mdd_stoch_grad(T(r), ti)
    lo, go = freq.batch_loss_grad(d, r, u, keep, nf)
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo
    assert abs(gn.item() - np.sum(go ** 2)) <= 2 * TOL * np.sum(go ** 2)


@pytest.mark.parametrize("nb", [3, 20, 40, 60])
def test_batch_of_rejected_entries_is_zero(nb):
    """No accepted entry: zero gradient and loss, also with kernel rows that are not finite."""
    d, u, r = random_case(70, 50, 35, 128, seed=nb)
    d[0] = np.inf
    plan = make_plan(d, u, nb_max=nb, nf=30)
    idx = T(np.full(nb, -1, dtype=np.int32), torch.int32)
    G, loss, gn = plan.mdd_stoch_grad(T(r), idx)
    assert not H(G).any() and loss.item() == 0.0 and gn.item() == 0.0


@pytest.mark.parametrize("prec,tol", [("fp32", TOL), ("bf16x3", 1e-3)])
@pytest.mark.parametrize("ns,nvs", [(64, 20), (130, 35), (130, 1), (193, 16)])
def test_full_gradient_in_batches_of_64(prec, tol, ns, nvs):
    """More sources than one batch of 64, whatever nb_max: whole and ragged last batches."""
    from paper_2202_04486_amd.plan import Plan
    nr, nt, nf = 33, 128, 40
    d, u, r = random_case(ns, nr, nvs, nt, seed=ns + nvs)
    plan = Plan(ns, nr, nvs, nt, nf, 3, precision=prec, full_grad=True)
    plan.mdd_set_kernel(T(d))
    plan.mdd_set_data(T(u))
    G, loss, gn = plan.mdd_full_grad(T(r))
    lo, go = freq.batch_loss_grad(d, r, u, np.arange(ns), nf)
    assert relerr(H(G), go) <= tol
    assert abs(loss.item() - lo) <= tol * lo
    assert abs(gn.item() - np.sum(go ** 2)) <= 2 * tol * np.sum(go ** 2)


@pytest.mark.parametrize("nt", [128, 512, 1024])
@pytest.mark.parametrize("nr,nvs,nb", [(8, 16, 4), (33, 35, 9), (100, 20, 7), (300, 1, 3), (300, 1, 40), (2000, 1, 17)])
def test_loss_and_norm_of_repeated_steps(nt, nr, nvs, nb):
    """The reductions at sizes where the update kernel's last workgroup does them and where a
    launch of its own does, repeated on one plan: every call's loss and gradient norm."""
    ns, nf = 45, 30
    d, u, r = random_case(ns, nr, nvs, nt, seed=nr + nb)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    rng = np.random.default_rng(nt)
    for _ in range(4):
        idx = rng.integers(0, ns, size=nb).astype(np.int32)
        lo, go = freq.batch_loss_grad(d, r, u, idx, nf)
        G, loss, gn = plan.mdd_stoch_grad(T(r), T(idx, torch.int32))
        assert relerr(H(G), go) <= TOL
        assert abs(loss.item() - lo) <= TOL * lo
        assert abs(gn.item() - np.sum(go ** 2)) <= 2 * TOL * np.sum(go ** 2)
        v = f32(rng.standard_normal((nb, nvs, nt)))
        assert relerr(H(plan.mdc_adjoint(T(v), T(idx, torch.int32))), freq.mdc_adjoint(d[idx], v, nf)) <= TOL


@pytest.mark.parametrize("nb", [1, 8, 9, 16, 17, 24, 25, 32, 33, 48, 64])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 48, 65, 321])
def test_products_with_reciprocity(n, nb):
    """The average in the products: row blocks shared by the two halves of the adjoint, mirrored
    entries of ragged chunks.  What an earlier call with a model that is not finite left in the
    plan's spectra must not come through."""
    ns, nt, nf = 66, 128, 33
    d, u, r = random_case(ns, n, n, nt, seed=n + nb)
    rng = np.random.default_rng(nb)
    idx = rng.integers(0, ns, size=nb).astype(np.int32)
    if nb > 4:
        idx[1], idx[nb - 1] = -1, ns
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    good = (idx >= 0) & (idx < ns)
    keep, ti = idx[good], T(idx, torch.int32)
    plan.mdd_stoch_grad(torch.full((n, n, nt), np.inf, device="cuda"), ti)
    mean = lambda z: 0.5 * (z + np.swapaxes(z, 0, 1))
    ug = H(plan.mdc_forward_rec(T(r), ti))
    assert relerr(ug[good], freq.mdc(d[keep], mean(r.astype(np.float64)), nf)) <= TOL
    assert not ug[~good].any()
    v = f32(rng.standard_normal((nb, n, nt)))
    v[~good] = np.nan
    ga = H(plan.mdc_adjoint_rec(T(v), ti))
    assert relerr(ga, mean(freq.mdc_adjoint(d[keep], v[good], nf))) <= TOL


# Bound per product and operand pair, relative to the norm: float32 spectra as above plus, for
# bf16x3, the rounding of two low halves and the dropped low * low term (3 * 2^-18); for
# fp16x3 the same at 2^-22; for bf16 the rounding of the two operands (2 * 2^-9).  The gradient
# and the loss go through a residual of such products: twice that.
SPLIT_TOL = {"bf16x3": TOL + 3 * 2.0 ** -18, "fp16x3": TOL + 3 * 2.0 ** -22, "bf16": TOL + 2.0 ** -8}


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3", "bf16"])
@pytest.mark.parametrize("nb,nr,nvs", [(1, 1, 2), (3, 33, 17), (16, 32, 65), (16, 321, 33), (17, 95, 64),
                                       (32, 64, 130), (33, 63, 18), (48, 65, 66), (49, 129, 20),
                                       (64, 40, 81)])
def test_every_split_kind_at_tile_edges(prec, nb, nr, nvs):
    ns, nt, nf, tol = 70, 128, 41, SPLIT_TOL[prec]
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb + nr + nvs)
    rng = np.random.default_rng(nb)
    idx = rng.integers(0, ns, size=nb).astype(np.int32)
    if nb > 4:
        idx[1], idx[nb - 1] = -1, ns
        idx[3] = idx[2]
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision=prec)
    good = (idx >= 0) & (idx < ns)
    keep, ti = idx[good], T(idx, torch.int32)
    plan.mdd_stoch_grad(torch.full((nr, nvs, nt), np.inf, device="cuda"), ti)  # leaves nothing behind
    out = torch.full((nb, nvs, nt), np.nan, device="cuda")
    ug = H(plan.mdc_forward(T(r), ti, out=out))
    assert relerr(ug[good], freq.mdc(d[keep], r, nf)) <= tol
    assert not ug[~good].any()
    v = f32(rng.standard_normal((nb, nvs, nt)))
    v[~good] = np.nan
    ga = H(plan.mdc_adjoint(T(v), ti))
    assert relerr(ga, freq.mdc_adjoint(d[keep], v[good], nf)) <= tol
    G, loss, gn = plan.mdd_stoch_grad(T(r), ti)
    lo, go = freq.batch_loss_grad(d, r, u, keep, nf)
    assert relerr(H(G), go) <= 2 * tol
    assert abs(loss.item() - lo) <= 2 * tol * lo
    assert abs(gn.item() - np.sum(go ** 2)) <= 4.1 * tol * np.sum(go ** 2)
    first = G.clone()
    for _ in range(4):
        assert torch.equal(plan.mdd_stoch_grad(T(r), ti)[0], first)


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3"])
@pytest.mark.parametrize("nf,nvs", [(63, 250), (64, 250), (33, 17)])
@pytest.mark.parametrize("nb,nr", [(9, 31), (20, 33), (40, 65), (64, 97)])
def test_split_products_with_few_and_many_workgroups(prec, nf, nvs, nb, nr):
    """Both sides of 256 workgroups (four column blocks each): one or two wavefronts per block,
    with odd and even numbers of receiver chunks."""
    ns, nt, tol = 70, 128, SPLIT_TOL[prec]
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb + nr)
    idx = np.random.default_rng(nb).integers(0, ns, size=nb).astype(np.int32)
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision=prec)
    ti = T(idx, torch.int32)
    assert relerr(H(plan.mdc_forward(T(r), ti)), freq.mdc(d[idx], r, nf)) <= tol
    G, loss, _ = plan.mdd_stoch_grad(T(r), ti)
    lo, go = freq.batch_loss_grad(d, r, u, idx, nf)
    assert relerr(H(G), go) <= 2 * tol
    assert abs(loss.item() - lo) <= 2 * tol * lo


@pytest.mark.parametrize("s,r", [(0, 0), (85, 40), (149, 89), (136, 63)])
def test_fp16_scale_finds_the_largest_entry_anywhere(s, r):
    """One trace 2^20 times the others: were it missed in the scale, its halves would overflow."""
    ns, nr, nvs, nt, nf = 150, 90, 20, 128, 30
    d, u, m = random_case(ns, nr, nvs, nt, seed=s)
    d[s, r] *= 2.0 ** 20
    plan = make_plan(d, u, nb_max=8, nf=nf, precision="fp16x3")
    idx = np.array([s, (s + 1) % ns], dtype=np.int32)
    G, loss, _ = plan.mdd_stoch_grad(T(m), T(idx, torch.int32))
    lo, go = freq.batch_loss_grad(d, m, u, idx, nf)
    assert relerr(H(G), go) <= 2 * SPLIT_TOL["fp16x3"]
    assert abs(loss.item() - lo) <= 2 * SPLIT_TOL["fp16x3"] * lo
