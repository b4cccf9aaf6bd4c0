"""fp16x3 at up to 16 batch rows: D's scales come from the batch, so a source outside it that
is far stronger, or not finite, costs the batch no bits."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, f32, make_plan, random_case, relerr

pytestmark = pytest.mark.gpu

# relative to the norm: float32 spectra (2e-6), the rounding of two low halves and the dropped
# low * low term (3 * 2^-22); the gradient goes through a residual of such products: twice that
TOL = 2e-6 + 3 * 2.0 ** -22


@pytest.mark.parametrize("weak,strong", [(1.0, 2.0 ** 22), (2.0 ** -16, 2.0 ** 126)])
@pytest.mark.parametrize("nb,nr,nvs,nf", [(1, 17, 3, 20), (5, 300, 35, 20), (16, 97, 250, 40), (9, 257, 250, 65)])
def test_strong_source_outside_the_batch(nb, nr, nvs, nf, weak, strong):
    ns, nt = 20, 128
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb + nr)
    d *= weak
    d[7] *= strong / weak                     # 2^126: its spectra overflow at some frequencies
    rng = np.random.default_rng(nb)
    idx = rng.choice([s for s in range(ns) if s != 7], size=nb, replace=False).astype(np.int32)
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision="fp16x3")
    ti = T(idx, torch.int32)
    assert relerr(H(plan.mdc_forward(T(r), ti)), freq.mdc(d[idx], r, nf)) <= TOL
    v = f32(rng.standard_normal((nb, nvs, nt)))
    assert relerr(H(plan.mdc_adjoint(T(v), ti)), freq.mdc_adjoint(d[idx], v, nf)) <= TOL
    G, loss, _ = plan.mdd_stoch_grad(T(r), ti)
    lo, go = freq.batch_loss_grad(d, r, u, idx, nf)
    assert relerr(H(G), go) <= 2 * TOL
    assert abs(loss.item() - lo) <= 2 * TOL * lo


def test_weak_receivers_keep_their_bits():
    """Receivers 2^22 weaker than their neighbours: the adjoint scales each by its own."""
    ns, nr, nvs, nt, nf, nb = 12, 70, 20, 128, 20, 8
    d, u, _ = random_case(ns, nr, nvs, nt, seed=1)
    d[:, 1::2] *= 2.0 ** -22
    plan = make_plan(d, u, nb_max=nb, nf=nf, precision="fp16x3")
    idx = np.arange(nb, dtype=np.int32)
    v = f32(np.random.default_rng(2).standard_normal((nb, nvs, nt)))
    ga, go = H(plan.mdc_adjoint(T(v), T(idx, torch.int32))), freq.mdc_adjoint(d[idx], v, nf)
    assert relerr(ga[0::2], go[0::2]) <= TOL
    assert relerr(ga[1::2], go[1::2]) <= TOL
