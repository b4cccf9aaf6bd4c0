"""The reductions inside the update kernel: the same bits on every one of many repetitions, with
other work between them, for every number of workgroups a plan can have there."""
import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, make_plan, random_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [128, 1024])
@pytest.mark.parametrize("nr,nvs", [(1, 3), (7, 16), (64, 20), (128, 16), (250, 1), (2000, 1)])
def test_same_bits_every_time(nr, nvs, nt):
    ns, nf, nb = 20, 30, 5
    d, u, r = random_case(ns, nr, nvs, nt, seed=nr + nt)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    ga, gb = np.array([3, 1, 7, 7, 12]), np.array([5, 0, 19])
    idx, other = (T(g.astype(np.int32), torch.int32) for g in (ga, gb))
    n = 200
    loss, gn = (torch.zeros(2 * n, dtype=torch.float64, device="cuda") for _ in range(2))
    R, G = T(r), torch.empty(r.shape, device="cuda")
    for i in range(n):
        plan.mdd_stoch_grad(R, idx, G_out=G, loss_out=loss[2 * i:2 * i + 1], gnorm2_out=gn[2 * i:2 * i + 1])
        plan.mdd_stoch_grad(R, other, G_out=G, loss_out=loss[2 * i + 1:2 * i + 2],
                            gnorm2_out=gn[2 * i + 1:2 * i + 2])
    for j, g in ((0, ga), (1, gb)):
        assert torch.equal(loss[j::2], loss[j].expand(n)) and torch.equal(gn[j::2], gn[j].expand(n))
        lo, go = freq.batch_loss_grad(d, r, u, g, nf)
        assert abs(loss[j].item() - lo) <= 2e-6 * lo
        assert abs(gn[j].item() - np.sum(go ** 2)) <= 4e-6 * np.sum(go ** 2)
    assert H(G).any()


@pytest.mark.parametrize("nt", [128, 256, 512, 1024])
@pytest.mark.parametrize("blocks", [1, 64, 128, 129, 254, 256])
def test_a_norm_that_is_not_finite_leaves_nothing_behind(nt, blocks):
    """Both sides of the largest number of workgroups, and NaN and infinite norms between."""
    ns, nf, nb = 6, 20, 3
    nr = max(blocks // (2 if nt >= 512 else 1), 1)
    d, u, r = random_case(ns, nr, 16, nt, seed=nr + nt)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = torch.tensor([4, 0, 2], dtype=torch.int32, device="cuda")
    lo, go = freq.batch_loss_grad(d, r, u, np.array([4, 0, 2]), nf)
    for bad in (float("nan"), float("inf"), 3e38):
        assert not torch.isfinite(plan.mdd_stoch_grad(torch.full_like(T(r), bad), idx)[2]).item()
        _, loss, gn = plan.mdd_stoch_grad(T(r), idx)
        assert abs(loss.item() - lo) <= 2e-6 * lo
        assert abs(gn.item() - np.sum(go ** 2)) <= 4e-6 * np.sum(go ** 2)
