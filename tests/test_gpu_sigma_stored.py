"""The power iteration between steps of a plan that stores the model's spectra: they survive
it, in eager steps and in steps captured to start from them."""
import ctypes

import pytest
import torch

from paper_2202_04486_amd import native
from gpu_helpers import T, batch, random_case


pytestmark = pytest.mark.gpu


def make(full, d, u, nb, nf):
    from paper_2202_04486_amd.plan import Plan
    ns, nr, nt = d.shape
    plan = Plan(ns, nr, u.shape[1], nt, nf, nb, store_rf=True, full_grad=full)
    plan.mdd_set_kernel(T(d))
    plan.mdd_set_data(T(u))
    return plan


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("nvs", [1, 35])
def test_no_second_model_transform(full, nvs):
    d, u, r = random_case(30, 33, nvs, 128, seed=3)
    idx = T(batch(30, 8, seed=1), torch.int32)
    plan = make(full, d, u, 8, 40)
    R, v = T(r), torch.zeros(r.shape, device="cuda")
    step = lambda: plan.mdd_full_step(R, opt="nsgd", lr=1e-7, s0=v) if full else \
        plan.mdd_step(R, idx, opt="nsgd", lr=1e-7, s0=v)
    step()
    plan.profile_enable(True, capacity=64)
    for _ in range(2):
        plan.mdd_sigma_max2(iters=3)
        step()
    assert plan.profile_read()["fft_model"][1] == 0


@pytest.mark.parametrize("nvs", [1, 35])
def test_captured_steps_that_start_from_stored_spectra(nvs):
    d, u, r = random_case(30, 33, nvs, 128, seed=4)
    idx = T(batch(30, 8, seed=1), torch.int32)
    plan = make(False, d, u, 8, 40)
    R, v = T(r), torch.zeros(r.shape, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    step = lambda: plan.mdd_step(R, idx, opt="nsgd", lr=1e-7, s0=v, loss_out=loss)

    def reset():
        R.copy_(T(r))
        v.zero_()
        plan.mdd_invalidate_model_spectra()

    want = []
    reset()
    for _ in range(4):
        step()
        want.append((R.clone(), loss.clone()))
    reset()
    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for rep in range(1, 4):
        g.replay()
        assert torch.equal(R, want[rep][0]) and torch.equal(loss, want[rep][1]), rep
        plan.mdd_sigma_max2(iters=2)
        torch.cuda.synchronize()


def test_static_workspace_takes_what_it_took():
    """The scratch of a plan that stores spectra is not asked of the static workspace of
    mdd_stoch_grad_noalloc, which runs no power iteration."""
    nr, nvs, nt, nf, nb = 64, 1, 256, 100, 8
    dims = lambda ns, flags: native.make_dims(ns, nr, nvs, nt, nf, nb, "fp32", flags)
    ns = max(n for n in range(64, 2000) if native.workspace_bytes(dims(n, 0)) <= native.NOALLOC_WORKSPACE_BYTES)
    assert native.workspace_bytes(dims(ns, native.FLAG_STORE_RF)) > native.NOALLOC_WORKSPACE_BYTES
    d, u, r = (torch.randn(s, device="cuda") for s in ((ns, nr, nt), (ns, nvs, nt), (nr, nvs, nt)))
    idx = torch.arange(nb, dtype=torch.int32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    out = []
    for flags in (0, native.FLAG_STORE_RF):
        G = torch.full_like(r, float("nan"))
        dm = dims(ns, flags)
        native.check("mdd_stoch_grad_noalloc", native.load().mdd_stoch_grad_noalloc(
            ctypes.byref(dm), p(d), p(u), None, p(r), p(idx), nb, p(G), None, None,
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        out.append(G)
    torch.cuda.synchronize()
    assert torch.isfinite(out[0]).all() and torch.equal(*out)
