"""Float32 products at up to 16 batch rows with few column blocks, where the wavefronts of a
workgroup share a block: both sides of the rule, chunks of receivers that fill some wavefronts,
all of D in LDS or two chunks of it, and the sum over batches."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, f32, make_plan, random_case, relerr

pytestmark = pytest.mark.gpu

TOL = 2e-6  # float32 spectra; the compensated products add less


@pytest.mark.parametrize("prec", ["fp32", "fp32_cgemm"])
@pytest.mark.parametrize("nb", [1, 6, 16])
@pytest.mark.parametrize("nr,nvs,nf", [(1, 2, 65), (32, 40, 65), (33, 40, 65), (40, 63, 64), (40, 65, 64), (128, 64, 65), (129, 64, 65),
                                       (160, 17, 33), (257, 33, 9), (384, 16, 20), (385, 20, 20), (416, 2, 30),
                                       (513, 48, 10), (140, 256, 64), (140, 257, 65)])
def test_shared_blocks(prec, nb, nr, nvs, nf):
    ns, nt = 18, 128
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
    assert relerr(ug[good], freq.mdc(d[keep], r, nf)) <= TOL
    assert not ug[~good].any()
    v = f32(rng.standard_normal((nb, nvs, nt)))
    v[~good] = np.nan
    assert relerr(H(plan.mdc_adjoint(T(v), ti)), freq.mdc_adjoint(d[keep], v[good], nf)) <= TOL
    G, loss, gn = plan.mdd_stoch_grad(T(r), ti)
    lo, go = freq.batch_loss_grad(d, r, u, keep, nf)
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo
    assert abs(gn.item() - np.sum(go ** 2)) <= 2 * TOL * np.sum(go ** 2)
    for _ in range(3):
        assert torch.equal(plan.mdd_stoch_grad(T(r), ti)[0], G)


@pytest.mark.parametrize("nr", [100, 230, 400])
def test_shared_blocks_add_to_the_full_gradient(nr):
    """A last batch of 9 rows on top of one of 64."""
    from paper_2202_04486_amd.plan import Plan
    ns, nvs, nt, nf = 73, 20, 128, 40
    d, u, r = random_case(ns, nr, nvs, nt, seed=nr)
    plan = Plan(ns, nr, nvs, nt, nf, 3, full_grad=True)
    plan.mdd_set_kernel(T(d))
    plan.mdd_set_data(T(u))
    G, loss, _ = plan.mdd_full_grad(T(r))
    lo, go = freq.batch_loss_grad(d, r, u, np.arange(ns), nf)
    assert relerr(H(G), go) <= TOL
    assert abs(loss.item() - lo) <= TOL * lo
