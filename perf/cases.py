"""The work this library is used for, as timed cases.

Every case is one call, or the few calls that belong together, through the package's
public entry points: a stochastic step (`Plan.mdd_step`), a mini-batch gradient
(`Plan.mdd_stoch_grad`), an epoch of the solver (`StochasticMDD.run_epoch`), a gradient
through torch.autograd (`mdc_rec`), a full-gradient iteration (`Plan.mdd_full_step`), a
new kernel with its step size (`Plan.mdd_set_kernel`, `Plan.mdd_sigma_max2`) and a step
on staged kernel and data rows (`Plan.mdd_stage_kernel`, `Plan.mdd_stage_data`).

Wavefields are sums of hyperbolic Ricker events over a line or a square grid of
receivers, drawn from the seed.  Models and optimiser states are those of a run that is
under way: a partly recovered model, moments at the scale of the gradient.

The float64 loss of a step is a sum over float32 residuals, of which about seven digits
mean anything, so it is returned as float32 where the host has it anyway (an epoch).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2202_04486_amd.autograd import mdc_rec
from paper_2202_04486_amd.plan import Plan
from paper_2202_04486_amd.solver import StochasticMDD

DT = 0.004          # sample interval (s)
V_MASK = 2500.0     # largest velocity of the reflections (m/s)
SIGMA_ITERS = 100   # the solver's default number of power iterations
BETA1, BETA2, EPS, MU = 0.9, 0.999, 1e-8, 0.9
LR_ADAM = 1e-3
T0 = 40             # steps already taken


def listed():
    line = dict(ns=201, nr=201, nvs=201, nt=1024, nf=257, grid=0)
    diff = dict(ns=301, nr=301, nvs=301, nt=1024, nf=257, grid=0, precision="fp32")
    patch = dict(ns=1600, nr=1600, nvs=1600, nt=512, nf=200, grid=40)
    return [
        # a toy line while a workflow is set up: launches and latency
        dict(name="tiny2d_step", op="step", ns=32, nr=32, nvs=32, nt=128, nf=65, grid=0, nb=8,
             precision="fp32", opt="sgd", mask=False),
        # the 2D line example: one step of the inversion
        dict(name="line2d_step", op="step", **line, nb=16, precision="fp32", opt="adam", mask=True),
        # the gradient alone at the ocean-bottom example's batch, for a caller's own optimiser
        dict(name="line2d_grad", op="grad", **line, nb=32, precision="fp32", mask=True),
        # the full-gradient (Landweber) baseline on the line; the plan also serves batches of 16
        dict(name="line2d_full_step", op="full", **line, nb=16, precision="fp32", opt="sgd",
             mask=True),
        # a new kernel and the step size that it allows
        dict(name="line2d_stepsize", op="stepsize", **line, nb=16, precision="fp32"),
        # one virtual source of the line: a whole epoch of Nesterov steps
        dict(name="line2d_vs1_epoch", op="epoch", **{**line, "nvs": 1}, nb=32, precision="fp32",
             opt="nsgd", mask=True),
        # one virtual source of the 3D patch
        dict(name="patch3d_vs1_step", op="step", **{**patch, "nvs": 1}, nb=64, precision="fp32",
             opt="adam", mask=True),
        # a loss in torch on the differentiable operator with reciprocity: small and ordinary batch
        dict(name="diff301_b8", op="diff", **diff, nb=8),
        dict(name="diff301_b32", op="diff", **diff, nb=32),
        # a 20 x 20 patch under many sources: kernel and data rows staged batch by batch
        dict(name="stream_step", op="stream", ns=3200, nr=400, nvs=400, nt=512, nf=200, grid=20,
             nb=48, precision="fp16x3", opt="nsgd", mask=True),
        # the 3D patch, the largest problem: in float32 and in the split form
        dict(name="patch3d_step", op="step", **patch, nb=64, precision="fp32", opt="adam", mask=True),
        dict(name="patch3d_step_bf16x3", op="step", **patch, nb=64, precision="bf16x3", opt="adam",
             mask=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "grad", "grad", "vs1", "epoch", "diff", "diff", "full",
                     "stepsize", "stream"])
    top = {"step": 1300, "grad": 900, "vs1": 2600, "epoch": 700, "diff": 420, "full": 420,
           "stepsize": 500, "stream": 500}[op]
    n = _log_int(rng, 24, top)

    def near():
        return max(16, min(top, int(n * rng.uniform(0.8, 1.2))))

    nt = rng.choice([128, 256, 512, 1024] if n <= 500 else [256, 512])
    c = dict(op=op, ns=near(), nr=near(), nvs=near(), nt=nt, nf=rng.randint(nt // 8, nt // 2 + 1), grid=0,
             nb=_log_int(rng, 1, 64), precision=rng.choice(["fp32", "fp32", "fp32", "bf16x3", "fp16x3"]))
    if op in ("step", "vs1", "epoch", "full", "stream"):
        c["opt"] = rng.choice(["adam", "sgd", "nsgd"] if n <= 500 and op != "epoch" else
                              ["sgd", "nsgd"] if op == "epoch" else ["adam"])
    if op not in ("diff", "stepsize"):
        c["mask"] = rng.random() < 0.7
    if op == "diff":
        c["nvs"] = c["nr"]
    if op == "vs1":
        c.update(op="step", nvs=1)
    if op == "epoch":
        c.update(nvs=1 if rng.random() < 0.6 else min(c["nvs"], 64),
                 nb=min(64, max(c["nb"], math.ceil(c["ns"] / 16))))
    if op == "stream":
        c["ns"] = _log_int(rng, 64, 5000)
    c["nb"] = min(c["nb"], c["ns"])
    return c


# ----------------------------------------------------------------- inputs
def _positions(n, grid, dev):
    i = torch.arange(n, device=dev, dtype=torch.float64)
    if grid:
        return torch.stack([i % grid, torch.div(i, grid, rounding_mode="floor")], 1) * 25.0
    return torch.stack([i, torch.zeros_like(i)], 1) * 10.0


def _h2(src, rec):
    return (src[:, None, 0] - rec[None, :, 0]) ** 2 + (src[:, None, 1] - rec[None, :, 1]) ** 2


def _cube(src, rec, nt, events, f0):
    """Sum of hyperbolic Ricker events [len(src)][len(rec)][nt], float32."""
    dev = src.device
    out = torch.empty((src.shape[0], rec.shape[0], nt), dtype=torch.float32, device=dev)
    t = torch.arange(nt, device=dev, dtype=torch.float32) * DT
    step = max(1, (1 << 26) // (rec.shape[0] * nt))
    for r0 in range(0, src.shape[0], step):
        h2 = _h2(src[r0:r0 + step], rec)
        part = out[r0:r0 + step]
        part.zero_()
        for t0, v, amp in events:
            arr = torch.sqrt(t0 * t0 + h2 / (v * v)).to(torch.float32)
            a = (t - arr[:, :, None]).mul_(math.pi * f0).square_()
            part += (1.0 - 2.0 * a).mul_(torch.exp(a.neg_())).mul_(amp)
    return out


def _inputs(case, seed):
    """What a program has in hand: wavefields, batch, model, optimiser state, mask."""
    dev = torch.device("cuda", torch.cuda.current_device())
    rng = np.random.default_rng([int(seed), case["ns"], case["nr"], case["nvs"], case["nt"]])
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(rng.integers(1 << 40)))
    ns, nr, nvs, nt, nb = (case[k] for k in ("ns", "nr", "nvs", "nt", "nb"))
    grid, op = case["grid"], case["op"]
    span = nt * DT
    f0 = 12.0 if grid else 15.0

    def events(n, lo, hi):
        return [(float(rng.uniform(lo * span, hi * span)), float(rng.uniform(1500.0, 2500.0)),
                 float(rng.choice([-1.0, 1.0]) * rng.uniform(0.5, 1.0))) for _ in range(n)]

    rec = _positions(nr, grid, dev)
    vs = rec[nr // 2:nr // 2 + 1] if nvs == 1 else _positions(nvs, grid, dev)
    idx = np.sort(rng.choice(ns, size=nb, replace=False)).astype(np.int32)
    # periodic down-going train, as under a free surface
    t1, period, vel = rng.uniform(0.03, 0.08) * span, rng.uniform(0.06, 0.1) * span, rng.uniform(1500.0, 2500.0)
    down = [(float(t1 + k * period), float(vel), (-0.6) ** k) for k in range(4)]
    src_all = _positions(ns, grid if ns <= nr else int(math.ceil(math.sqrt(ns))) if grid else 0, dev)
    if grid == 0 and ns > nr:   # more sources than receivers: the same line, denser
        src_all = src_all * (nr / ns)
    src = src_all[torch.from_numpy(idx).long().to(dev)] if op == "stream" else src_all
    x = {"idx": idx, "d": _cube(src, rec, nt, down, f0)}
    if op == "stepsize":
        return x
    x["u"] = _cube(src, vs, nt, events(3, 0.1, 0.6), f0)
    scale = math.sqrt(nr * nt) * float(x["d"][:8].double().square().mean().sqrt())
    x["u"] *= 0.1 * scale     # the scale of the operator's output for the model below
    r = _cube(rec, vs, nt, events(3, 0.08, 0.4), f0).mul_(0.3)
    step = max(1, (1 << 26) // (nvs * nt))
    for r0 in range(0, nr, step):
        r[r0:r0 + step] += torch.randn(r[r0:r0 + step].shape, generator=gen, device=dev) * 0.01
    onset = None
    if case.get("mask"):
        onset = torch.ceil((_h2(rec, vs).sqrt() / V_MASK - 1.5 / f0) / DT).clamp_(0, nt // 2).to(torch.int32)
        t = torch.arange(nt, device=dev, dtype=torch.int32)
        for r0 in range(0, nr, step):
            r[r0:r0 + step] *= t >= onset[r0:r0 + step, :, None]
    x["R"], x["onset"] = r, onset
    opt = case.get("opt")
    if opt == "adam":         # moments at the scale of the gradient
        g = (math.sqrt(nb * nt) * float(x["d"][:8].double().square().mean().sqrt())
             * float(x["u"][:8].double().square().mean().sqrt()))
        x["s0"] = torch.empty_like(r).normal_(generator=gen).mul_(0.3 * g)
        x["s1"] = torch.empty_like(r).uniform_(0.05, 1.0, generator=gen).mul_(g * g)
        x["lr"] = LR_ADAM
    elif opt:                 # a step size that any batch is stable under
        f = torch.zeros(case["nf"], dtype=torch.float64, device=dev)
        for s0 in range(0, x["d"].shape[0], 32):
            z = torch.fft.rfft(x["d"][s0:s0 + 32], dim=-1)[..., :case["nf"]]
            f += (z.real.double().square() + z.imag.double().square()).sum((0, 1))
        x["lr"] = 0.5 / float(f.max())
        if opt == "nsgd":
            x["s0"] = r * (torch.randn((nr, nvs, 1), generator=gen, device=dev) * 0.02)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    dev = x["d"].device
    plan = Plan(case["ns"], case["nr"], case["nvs"], case["nt"], case["nf"], case["nb"],
                precision=case["precision"], store_rf=op in ("step", "epoch", "full", "stream"),
                full_grad=op == "full", stream_kernel=op == "stream", stream_data=op == "stream")
    st = {"op": op, "plan": plan, "idx": torch.from_numpy(x["idx"]).to(dev), "t": T0, "case": dict(case)}
    if op == "stepsize":
        st["d"] = x["d"]
        return st
    if op == "stream":
        st["d_rows"], st["u_rows"] = x["d"], x["u"]
    else:
        plan.mdd_set_kernel(x["d"])
        if op != "diff":
            plan.mdd_set_data(x["u"])
    if x["onset"] is not None:
        plan.mdd_set_mask(x["onset"])
    if op == "diff":
        st["z"] = x["R"].requires_grad_(True)
        st["ub"] = x["u"][st["idx"].long()].contiguous()
        return st
    st["R"] = x["R"]
    if op == "grad":
        return st
    st["opt"], st["lr"] = case["opt"], x["lr"]
    st["s0"], st["s1"] = x.get("s0"), x.get("s1")
    st["loss"] = torch.zeros(1, dtype=torch.float64, device=dev)
    st["gn"] = torch.zeros(1, dtype=torch.float64, device=dev)
    if op == "epoch":
        sol = StochasticMDD(plan, optimizer=case["opt"], lr=x["lr"], nb=case["nb"], mu=MU, R0=x["R"])
        if sol.s0 is not None:
            sol.s0.copy_(x["s0"])
        st["solver"] = sol
        st["perm"] = _perm(case, seed)
    torch.cuda.synchronize()
    return st


def _perm(case, seed):
    return np.random.default_rng([int(seed), 7]).permutation(case["ns"])


def run(state):
    op, plan = state["op"], state["plan"]
    if op == "grad":
        return {"G": plan.mdd_stoch_grad(state["R"], state["idx"])[0]}
    if op == "diff":
        z = state["z"]
        z.grad = None
        pred = mdc_rec(z, state["idx"], plan)
        loss = 0.5 * (pred - state["ub"]).square().sum()
        loss.backward()
        return {"U": pred.detach(), "grad": z.grad, "loss": loss.detach()}
    if op == "stepsize":
        plan.mdd_set_kernel(state["d"])
        return {"lam": plan.mdd_sigma_max2(iters=SIGMA_ITERS).float()}
    if op == "epoch":
        sol = state["solver"]
        loss = sol.run_epoch(state["perm"])
        out = {"R": sol.R, "loss": loss.astype(np.float32)}
        if sol.s0 is not None:
            out["s0"] = sol.s0
        return out
    R, s0, s1 = state["R"], state["s0"], state["s1"]
    state["t"] += 1
    if op == "full":
        plan.mdd_full_step(R, opt=state["opt"], lr=state["lr"], s0=s0, s1=s1, t=state["t"], beta1=BETA1,
                           beta2=BETA2, eps=EPS, mu=MU, loss_out=state["loss"], gnorm2_out=state["gn"])
    else:
        if op == "stream":
            plan.mdd_stage_kernel(state["d_rows"])
            plan.mdd_stage_data(state["u_rows"])
        plan.mdd_step(R, state["idx"], opt=state["opt"], lr=state["lr"], s0=s0, s1=s1, t=state["t"],
                      beta1=BETA1, beta2=BETA2, eps=EPS, mu=MU, loss_out=state["loss"],
                      gnorm2_out=state["gn"])
    out = {"R": R}
    if state["opt"] in ("adam", "nsgd"):
        out["s0"] = s0
    if state["opt"] == "adam":
        out["s1"] = s1
    return out


# ----------------------------------------------------------------- what a pass cannot do without
def work(case):
    ns, nr, nvs, nt, nf, nb = (case[k] for k in ("ns", "nr", "nvs", "nt", "nf", "nb"))
    op = case["op"]
    model, fft = 4 * nr * nvs * nt, 2.5 * nt * math.log2(nt)
    if op == "stepsize":
        return {"bytes": 4 * ns * nr * nt + 4 * nf,
                "flops": ns * nr * fft + 16 * ns * nr * nf * SIGMA_ITERS}
    if op == "diff":      # z in, gradient out; forward and adjoint products
        return {"bytes": 2 * model + 8 * nb * nr * nf + 8 * nb * nvs * nt,
                "flops": 16 * nb * nr * nvs * nf + 2 * (nr + nb) * nvs * fft}
    mask = 4 * nr * nvs if case.get("mask") else 0
    if op == "grad":
        return {"bytes": 2 * model + mask + 8 * nb * (nr + nvs) * nf,
                "flops": 16 * nb * nr * nvs * nf + 2 * nr * nvs * fft}
    state = model * 2 * {"sgd": 1, "nsgd": 2, "adam": 3}[case["opt"]]
    if op == "epoch":
        steps = math.ceil(ns / nb)
        return {"bytes": steps * (state + mask) + 8 * ns * (nr + nvs) * nf,
                "flops": 16 * ns * nr * nvs * nf + 2 * steps * nr * nvs * fft}
    rows = ns if op == "full" else nb
    data = 4 * nb * (nr + nvs) * nt if op == "stream" else 8 * rows * (nr + nvs) * nf
    more = nb * (nr + nvs) * fft if op == "stream" else 0
    return {"bytes": state + mask + data, "flops": 16 * rows * nr * nvs * nf + 2 * nr * nvs * fft + more}


# ----------------------------------------------------------------- the same in 64 bits
def _spectra(x, nf):
    """[rows][cols][nt] -> [nf][rows][cols] complex128."""
    out = torch.empty((nf, x.shape[0], x.shape[1]), dtype=torch.complex128, device=x.device)
    step = max(1, (1 << 25) // (x.shape[1] * x.shape[2]))
    for r0 in range(0, x.shape[0], step):
        out[:, r0:r0 + step] = torch.fft.rfft(x[r0:r0 + step].double(), dim=-1)[..., :nf].permute(2, 0, 1)
    return out


def _traces(spec, nt):
    """[nf][rows][cols] complex128 -> [rows][cols][nt] float64."""
    out = torch.empty((spec.shape[1], spec.shape[2], nt), dtype=torch.float64, device=spec.device)
    step = max(1, (1 << 25) // (spec.shape[2] * nt))
    for r0 in range(0, spec.shape[1], step):
        out[r0:r0 + step] = torch.fft.irfft(spec[:, r0:r0 + step].permute(1, 2, 0).contiguous(), n=nt, dim=-1)
    return out


def _outside(u, nf):
    """Energy of the rows of u in the bins that are not retained, [rows]."""
    z = torch.fft.rfft(u.double(), dim=-1)
    nt = u.shape[-1]
    w = torch.full((z.shape[-1],), 2.0, dtype=torch.float64, device=u.device)
    w[0] = w[-1] = 1.0
    w[:nf] = 0.0
    return ((z.real ** 2 + z.imag ** 2) * w).sum((1, 2)) / (2.0 * nt)


def _gradient(model, dk, uk, nf, nt):
    """Time-domain gradient at `model` and the in-band loss, for the rows dk, uk [nf][nb][.]."""
    rk = _spectra(model, nf)
    loss = 0.0
    w = torch.full((nf,), 2.0, dtype=torch.float64, device=model.device)
    w[0] = 1.0
    if 2 * (nf - 1) == nt:
        w[-1] = 1.0
    for k in range(nf):
        res = torch.matmul(dk[k], rk[k]) - uk[k]
        loss = loss + w[k] * (res.real ** 2 + res.imag ** 2).sum()
        rk[k] = torch.matmul(dk[k].conj().t().contiguous(), res)
    return _traces(rk, nt), float(loss) / (2.0 * nt)


def _muted(x, onset):
    if onset is None:
        return x
    t = torch.arange(x.shape[-1], device=x.device, dtype=torch.int32)
    step = max(1, (1 << 26) // (x.shape[1] * x.shape[2]))
    for r0 in range(0, x.shape[0], step):
        x[r0:r0 + step] *= t >= onset[r0:r0 + step, :, None]
    return x


def _sigma(dk, iters):
    r = torch.arange(dk.shape[2], device=dk.device)
    v = torch.complex(1.0 + 0.25 * ((r * 37) % 11).double(), 0.1 * ((r * 17) % 7).double())
    v = (v / torch.linalg.vector_norm(v)).expand(dk.shape[0], -1).unsqueeze(-1).contiguous()
    dh = dk.conj().transpose(1, 2).contiguous()
    lam = None
    for _ in range(iters):
        y = torch.matmul(dk, v)
        lam = (y.real ** 2 + y.imag ** 2).sum((1, 2))
        v = torch.matmul(dh, y)
        v = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
    return lam


def exact(case, seed):
    x = _inputs(case, seed)
    op, nf, nt = case["op"], case["nf"], case["nt"]
    d = x.pop("d")
    rows = torch.from_numpy(x["idx"]).long().to(d.device)
    if op == "stepsize":
        return {"lam": _sigma(_spectra(d, nf), SIGMA_ITERS)}
    u, onset = x.pop("u"), x["onset"]
    if op not in ("stream", "full", "epoch"):
        d, u = d[rows], u[rows]
    dk, uk = _spectra(d, nf), _spectra(u, nf)
    if op == "diff":
        z = x["R"].double()
        rk = _spectra(0.5 * (z + z.transpose(0, 1)), nf)
        pred = _traces(torch.matmul(dk, rk), nt)
        del rk
        res = pred - u.double()
        g = _traces(torch.matmul(dk.conj().transpose(1, 2).contiguous(), _spectra(res, nf)), nt)
        return {"U": pred, "grad": 0.5 * (g + g.transpose(0, 1)), "loss": 0.5 * res.square().sum()}
    if op == "grad":
        return {"G": _muted(_gradient(x["R"], dk, uk, nf, nt)[0], onset)}
    opt, lr = case["opt"], float(np.float32(x["lr"]))
    mu, b1, b2 = float(np.float32(MU)), float(np.float32(BETA1)), float(np.float32(BETA2))
    if op == "epoch":
        r = x["R"].double()
        v = x["s0"].double() if opt == "nsgd" else torch.zeros_like(r)
        m = mu if opt == "nsgd" else 0.0
        oob, losses = _outside(u, nf), []
        for b in batches_of(case, seed):
            b = torch.from_numpy(b).long().to(r.device)
            g, loss = _gradient(r + m * v, dk[:, b], uk[:, b], nf, nt)
            losses.append(loss + float(oob[b].sum()))
            v = _muted(m * v - lr * _muted(g, onset), onset)
            r = _muted(r + v, onset)
        out = {"R": r, "loss": np.array(losses)}
        if opt == "nsgd":
            out["s0"] = v
        return out
    R = x.pop("R")
    at = R.double() + mu * x["s0"].double() if opt == "nsgd" else R
    g = _muted(_gradient(at, dk, uk, nf, nt)[0], onset)
    del dk, uk, d, u, at
    if opt == "adam":
        s0, s1 = x.pop("s0").double().mul_(b1), x.pop("s1").double().mul_(b2)
        s0 += (1.0 - BETA1) * g
        s1 += (1.0 - BETA2) * g.square_()
        del g
        t = T0 + 1
        upd = (s1 / (1.0 - BETA2 ** t)).sqrt_().add_(EPS).reciprocal_().mul_(s0).mul_(-lr / (1.0 - BETA1 ** t))
        upd += R
        return {"R": _muted(upd, onset), "s0": s0, "s1": s1}
    if opt == "nsgd":
        v = _muted(mu * x["s0"].double() - lr * g, onset)
        return {"R": _muted(R.double() + v, onset), "s0": v}
    return {"R": _muted(R.double() - lr * g, onset)}


def batches_of(case, seed):
    """The batches of the epoch that run() takes: consecutive slices of the permutation."""
    perm, nb = _perm(case, seed), case["nb"]
    return [np.sort(perm[j:j + nb]) for j in range(0, len(perm), nb)]
