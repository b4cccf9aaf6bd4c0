"""The power iteration over all sources: rows held by one wavefront (up to 512 receivers, one
to four pairs a lane) and spread over several, ragged row groups, one iteration and more."""
import numpy as np
import pytest
import torch

from gpu_helpers import H, T, random_case

pytestmark = pytest.mark.gpu


def power_iteration(d, nf, iters):
    D = np.fft.rfft(d, axis=-1)[..., :nf].transpose(2, 0, 1)
    r = np.arange(d.shape[1])
    v = (1.0 + 0.25 * ((r * 37) % 11)) + 0.1j * ((r * 17) % 7)
    v = np.repeat((v / np.linalg.norm(v))[None, :, None], nf, axis=0)
    for _ in range(iters):
        y = D @ v
        lam = np.sum(np.abs(y) ** 2, axis=(1, 2))
        v = D.conj().transpose(0, 2, 1) @ y
        v /= np.linalg.norm(v, axis=1, keepdims=True)
    return lam


@pytest.mark.parametrize("iters", [1, 2, 9])
@pytest.mark.parametrize("ns,nr,nvs", [(1, 1, 1), (3, 1, 40), (17, 100, 1), (40, 128, 5), (33, 129, 20), (64, 256, 1),
                                       (70, 257, 70), (20, 512, 1), (21, 513, 3), (50, 1030, 33), (18, 2049, 1)])
def test_power_iteration_matches_numpy(ns, nr, nvs, iters):
    from paper_2202_04486_amd.plan import Plan
    nt, nf = 128, 11
    d, _, _ = random_case(ns, nr, 1, nt, seed=ns + nr)
    plan = Plan(ns, nr, nvs, nt, nf, 1)
    plan.mdd_set_kernel(T(d))
    lam = H(plan.mdd_sigma_max2(iters=iters))
    ref = power_iteration(d, nf, iters)
    # the float32 spectra carry up to about 1e-6 of relative rounding, lam twice that
    assert np.max(np.abs(lam - ref) / ref) <= 4e-6


def test_steps_after_a_power_iteration_are_unchanged():
    """Its scratch is the model spectra's buffer: stored spectra are taken again after it."""
    from gpu_helpers import batch, make_plan
    d, u, r = random_case(30, 33, 35, 128, seed=3)
    idx = T(batch(30, 8, seed=1), torch.int32)
    out = []
    for between in (False, True):
        plan = make_plan(d, u, nb_max=8, nf=40, store_rf=True)
        R, v = T(r), torch.zeros(r.shape, device="cuda")
        for t in range(3):
            plan.mdd_step(R, idx, opt="nsgd", lr=1e-7, s0=v)
            if between:
                plan.mdd_sigma_max2(iters=3)
        out.append(H(R))
    assert np.max(np.abs(out[0] - out[1])) <= 1e-6 * np.max(np.abs(out[0]))
