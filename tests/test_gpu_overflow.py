"""Four-product float32 sums that overflow are infinite, as plain sums are, and not NaN."""
import math

import pytest
import torch

from gpu_helpers import T, make_plan, random_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nb,nr", [("fp32", 3, 40), ("fp32", 16, 200), ("fp32_cgemm", 8, 33),
                                        ("fp32_cgemm", 8, 400), ("fp32_cgemm", 30, 70)])
def test_overflowing_loss_is_infinite(prec, nb, nr):
    ns, nvs, nt = 32, 20, 128
    d, u, r = random_case(ns, nr, nvs, nt, seed=nb)
    d[...] = r[...] = 0.0
    d[:, :, 0], r[:, :, 0] = 2.0 ** 70, 2.0 ** 60      # real spectra: no inf - inf in the products
    plan = make_plan(d, u, nb_max=nb, nf=40, precision=prec)
    _, loss, _ = plan.mdd_stoch_grad(T(r), torch.arange(nb, dtype=torch.int32, device="cuda"))
    assert loss.item() == math.inf
