"""Every instance of the split and bf16 products (1 to 4 blocks of batch rows; one wavefront or
two per column block; written, streamed or added to what is there): within its bound of the
oracle, and the same bits on every repetition."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, f32, make_plan, random_case, relerr

pytestmark = pytest.mark.gpu

# float32 spectra (2e-6) and the split of the two operands; twice through the residual
TOL = {"bf16x3": 2e-6 + 3 * 2.0 ** -18, "fp16x3": 2e-6 + 3 * 2.0 ** -22, "bf16": 2e-6 + 2.0 ** -8}


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3", "bf16"])
@pytest.mark.parametrize("nvs,nf", [(35, 40), (260, 60)])          # 40 and 300 workgroups
@pytest.mark.parametrize("rows", [9, 30, 48, 63])
def test_batches_added_to_the_full_gradient(prec, nvs, nf, rows):
    """A batch of 64 and one of 9 to 63 on top of it."""
    from paper_2202_04486_amd.plan import Plan
    ns, nr, nt = 64 + rows, 70, 128
    d, u, r = random_case(ns, nr, nvs, nt, seed=rows)
    plan = Plan(ns, nr, nvs, nt, nf, 4, precision=prec, full_grad=True)
    plan.mdd_set_kernel(T(d))
    plan.mdd_set_data(T(u))
    R = T(r)
    G, loss, _ = plan.mdd_full_grad(R)
    lo, go = freq.batch_loss_grad(d, r, u, np.arange(ns), nf)
    assert relerr(H(G), go) <= 2 * TOL[prec]
    assert abs(loss.item() - lo) <= 2 * TOL[prec] * lo
    for _ in range(20):
        g, l, _ = plan.mdd_full_grad(R)
        assert torch.equal(g, G) and torch.equal(l, loss)


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3", "bf16"])
@pytest.mark.parametrize("nvs,nf", [(35, 40), (260, 60)])
@pytest.mark.parametrize("nb", [9, 30, 48, 63])
def test_operators_and_gradient_repeat(prec, nvs, nf, nb):
    ns, nr, nt = 64, 70, 128
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb)
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision=prec)
    idx = np.random.default_rng(nb).integers(0, ns, size=nb).astype(np.int32)
    v = f32(np.random.default_rng(nb).standard_normal((nb, nvs, nt)))
    R, V, it = T(r), T(v), T(idx, torch.int32)
    calls = (lambda: plan.mdc_forward(R, it), lambda: plan.mdc_adjoint(V, it), lambda: plan.mdd_stoch_grad(R, it)[0])
    want = [c() for c in calls]
    for _ in range(20):
        assert all(torch.equal(c(), w) for c, w in zip(calls, want))
    assert relerr(H(want[0]), freq.mdc(d[idx], r, nf)) <= TOL[prec]
    assert relerr(H(want[1]), freq.mdc_adjoint(d[idx], v, nf)) <= TOL[prec]
    assert relerr(H(want[2]), freq.batch_loss_grad(d, r, u, idx, nf)[1]) <= 2 * TOL[prec]
