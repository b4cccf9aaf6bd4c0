"""The loss and the gradient norm are summed only where they are asked for."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import freq

from gpu_helpers import H, T, make_plan, random_case

pytestmark = pytest.mark.gpu


def sgd_step(plan, R, idx, lr, loss=None, gn=None):
    """One SGD step through the C ABI, where either scalar may be NULL."""
    from paper_2202_04486_amd import native
    p = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else 0)
    o = native.Opt(native.OPT["sgd"], 0, lr, 0.9, 0.999, 1e-8, 0.9, 1)
    plan._sync_stream()
    native.check("mdd_step", plan.lib.mdd_step(plan._plan, p(R), None, None, ctypes.byref(o), p(idx), idx.numel(),
                                               p(loss), p(gn)))


def captured_kernels(call):
    """Launches that `call` records into a HIP graph."""
    from paper_2202_04486_amd import native
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = ctypes.c_size_t(0)
    assert native.load().hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def test_long_norm_sums_cost_a_launch_only_where_asked_for():
    """34816 partials of the norm are summed in two launches, the 68 of the loss in one."""
    ns, nr, nvs, nt, nf, nb = 4, 2048, 257, 128, 4, 2
    d, u, _ = random_case(ns, nr, 1, nt, seed=1)
    u = np.repeat(u, nvs, axis=1)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = torch.arange(nb, dtype=torch.int32, device="cuda")
    R = torch.zeros((nr, nvs, nt), device="cuda")
    loss, gn = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
    neither = captured_kernels(lambda: sgd_step(plan, R, idx, 1e-9))
    assert captured_kernels(lambda: sgd_step(plan, R, idx, 1e-9, loss)) == neither + 1
    assert captured_kernels(lambda: sgd_step(plan, R, idx, 1e-9, loss, gn)) == neither + 2


@pytest.mark.parametrize("nr,nvs,nb", [(8, 16, 4), (40, 130, 9), (300, 1, 3), (300, 1, 40)])
def test_either_scalar_alone(nr, nvs, nb):
    """Both alone give what both together give, also after another call left its partials."""
    ns, nt, nf = 45, 128, 30
    d, u, r = random_case(ns, nr, nvs, nt, seed=nr + nb)
    plan = make_plan(d, u, nb_max=nb, nf=nf)
    idx = T(np.random.default_rng(nb).integers(0, ns, size=nb).astype(np.int32), torch.int32)
    out = []
    for want in ("lg", "l", "g", "", "lg"):
        loss, gn = (torch.full((1,), -1.0, dtype=torch.float64, device="cuda") for _ in range(2))
        R = T(r)
        sgd_step(plan, R, idx, 1e-6, loss if "l" in want else None, gn if "g" in want else None)
        out.append((loss.item(), gn.item(), R))
    (l, g, R), _, _, _, last = out
    assert l > 0 and g > 0 and (last[0], last[1]) == (l, g)
    assert out[1][:2] == (l, -1.0) and out[2][:2] == (-1.0, g) and out[3][:2] == (-1.0, -1.0)
    assert all(torch.equal(o[2], R) for o in out)
    lo, go = freq.batch_loss_grad(d, r, u, H(idx).astype(int), nf)
    assert abs(l - lo) <= 1e-5 * lo and abs(g - np.sum(go ** 2)) <= 2e-5 * np.sum(go ** 2)
