"""Performance cases of the library: what its users have it do, through the Python binding.

A case is a dict of plain values; ``prepare`` makes what a program holds before the call (the
medium, its tables and tallies, a network, a batch of samples), ``run`` is one call as such a
program makes it, ``work`` the bytes and operations one call cannot do without and ``exact``
the call's result in 64 bits where it has one.  Walks return exact integer tallies (with the
means and variances derived from them); their media differ from seed to seed by a few per cent
in opacity and by the Philox seed of the run.

Kinds of case:
  job     a new medium from the description to the results: tables, walk, read-back;
  walk    a medium whose tables are kept: one more run and its read-back;
  exit    a medium whose tables are kept: the exact exit kernel built for it, the walk with it
          and the read-back;
  data    training samples of the escape surrogate from a set of probe media;
  train   one optimiser step of the surrogate's network on one minibatch;
  attach  the network evaluated into the sampling records of a cloud.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1709_10187_amd import media, rddmc, surrogate

CLOUD = {"kind": "walk", "geometry": "slab", "clouds": 1, "tau0": 1.0e4, "T": 1.0e4, "cells": 64, "bins": 128,
         "grid": "uniform", "v_max": 0.0, "tau_th": 0.0, "groups": False, "dust": 0.0, "weights": False,
         "census": 0, "packets": 1 << 14}


def cloud(**kw):
    return {**CLOUD, **kw}


def cube(**kw):
    return {"kind": "job", "geometry": "cube", "n": 24, "bins": 256, "sigma_v": 20.0, "sources": 64,
            "packets": 1 << 16, **kw}


def listed():
    return [
        # the first call of any user, and the smoke check's: a small slab, solved from nothing
        cloud(name="slab_first_look", kind="job", tau0=300.0, cells=8, bins=16, packets=50000),
        # the tau0 = 1e5 slab of the method's own tests, plain rDDMC on the full uniform grid
        cloud(name="slab_tau1e5", tau0=1.0e5, packets=1 << 14),
        # a batch of small outflowing spheres of different depth, temperature, grid and velocity,
        # as a parameter study submits them
        cloud(name="outflow_batch", kind="job", geometry="sphere", clouds=8, tau0=3.0e3, cells=24, bins=64,
              v_max=60.0, packets=1 << 13),
        # the tau0 = 1e7 sphere on the paper's efficient frequency grid
        cloud(name="sphere_efficient", geometry="sphere", tau0=1.0e7, cells=256, bins=0, grid="efficient",
              packets=1 << 20),
        # the tau0 = 1e7 sphere on the full 256 x 512 grid with the exact exit kernel, time to
        # solution once its tables stand
        cloud(name="sphere_exit_kernel", kind="exit", geometry="sphere", tau0=1.0e7, cells=256, bins=512,
              packets=1 << 18),
        # time-dependent transport: a dusty slab with continuous-MC wings and census estimators
        cloud(name="slab_hybrid_census", tau0=1.0e4, bins=48, tau_th=10.0, dust=0.05, census=8, packets=1 << 14),
        # frequency-group Monte Carlo (the paper's Sec. 5.3), redistribution tables included
        cloud(name="slab_groups", kind="job", tau0=3.0e3, tau_th=media.ALL_THIN, groups=True, packets=1 << 14),
        # 3D hybrid transport through a lognormal cube: the grid of the full-size benchmark
        cube(name="cube_128", kind="walk", n=128, packets=1 << 22),
        # the same medium at the size of a quick study, from nothing
        cube(name="cube_24", n=24, packets=1 << 16),
        # the learned escape surrogate: data, an optimiser step, inference into a cloud's records
        {"name": "surrogate_data", "kind": "data", "probes": 256, "per_probe": 1024, "tau_max": 1.0e9},
        {"name": "surrogate_train", "kind": "train", "batch": 4096},
        {"name": "surrogate_attach", "kind": "attach", "clouds": 16, "tau0": 3.0e7, "T": 1.0e4, "cells": 256,
         "dx": 0.6, "v_max": 20.0, "max_batch": 4096},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _count(rng, lo, hi):
    return int(round(_log(rng, lo, hi)))


def _draw_plain(rng):
    geo = rng.choice(["slab", "sphere"])
    tau0 = _log(rng, 100.0, 5.0e4)
    return cloud(kind=rng.choice(["job", "walk"]), geometry=geo, tau0=tau0, T=_log(rng, 100.0, 5.0e4),
                 cells=_count(rng, 5, 96), bins=_count(rng, 16, 160),
                 v_max=rng.choice([0.0, _log(rng, 5.0, 150.0)]) if geo == "sphere" else 0.0,
                 packets=_count(rng, 1000, 60000))


def _draw_batch(rng):
    return cloud(kind=rng.choice(["job", "walk"]), geometry="sphere", clouds=rng.randint(2, 12),
                 tau0=_log(rng, 300.0, 1.0e4), T=_log(rng, 300.0, 3.0e4), cells=_count(rng, 8, 40),
                 bins=_count(rng, 24, 96), v_max=_log(rng, 10.0, 120.0), packets=_count(rng, 1000, 12000))


def _draw_efficient(rng):
    return cloud(geometry=rng.choice(["slab", "sphere"]), tau0=_log(rng, 1.0e6, 1.0e9), cells=_count(rng, 32, 256),
                 bins=0, grid="efficient", packets=_count(rng, 20000, 1 << 20))


def _draw_exit(rng):
    return cloud(kind="exit", geometry=rng.choice(["slab", "sphere"]), tau0=_log(rng, 1.0e6, 3.0e7),
                 cells=_count(rng, 32, 256), bins=_count(rng, 128, 512), packets=_count(rng, 10000, 1 << 18))


def _draw_hybrid(rng):
    dust = rng.choice([0.0, _log(rng, 0.01, 0.3)])
    return cloud(geometry=rng.choice(["slab", "sphere"]), tau0=_log(rng, 300.0, 5.0e3), T=_log(rng, 1.0e3, 3.0e4),
                 cells=_count(rng, 16, 64), bins=_count(rng, 24, 64), tau_th=rng.choice([5.0, 10.0, 20.0]),
                 dust=dust, weights=dust > 0.0 and rng.random() < 0.5, census=rng.choice([0, 4, 8]),
                 packets=_count(rng, 2000, 30000))


def _draw_groups(rng):
    return cloud(kind=rng.choice(["job", "walk"]), geometry=rng.choice(["slab", "sphere"]),
                 tau0=_log(rng, 300.0, 5.0e3), cells=_count(rng, 8, 64), bins=_count(rng, 48, 160),
                 tau_th=rng.choice([10.0, media.ALL_THIN]), groups=True, packets=_count(rng, 2000, 30000))


def _draw_cube(rng):
    return cube(kind=rng.choice(["job", "walk"]), n=_count(rng, 10, 64), bins=_count(rng, 48, 256),
                sigma_v=rng.choice([0.0, _log(rng, 5.0, 40.0)]), sources=_count(rng, 1, 64),
                packets=_count(rng, 5000, 400000))


def _draw_data(rng):
    return {"kind": "data", "probes": _count(rng, 32, 400), "per_probe": _count(rng, 200, 1500),
            "tau_max": _log(rng, 1.0e6, 1.0e9)}


def _draw_train(rng):
    return {"kind": "train", "batch": _count(rng, 100, 8192)}


def _draw_attach(rng):
    return {"kind": "attach", "clouds": rng.randint(1, 24), "tau0": _log(rng, 2.0e7, 5.0e8),
            "T": _log(rng, 500.0, 3.0e4), "cells": _count(rng, 32, 128), "dx": rng.uniform(0.6, 2.5),
            "v_max": rng.uniform(2.0, 25.0), "max_batch": rng.choice([1000, 4096, 10000])}


def draw(rng):
    return rng.choice([_draw_plain, _draw_batch, _draw_efficient, _draw_exit, _draw_hybrid, _draw_groups, _draw_cube,
                       _draw_data, _draw_train, _draw_attach])(rng)


# ---- media ------------------------------------------------------------------------------


def _medium(case, rng, scale):
    """One cloud of a case, its opacity jittered by a few per cent from the seed; the clouds of a
    batch also differ in temperature, grid and velocity."""
    tau0 = case["tau0"] * 10.0 ** rng.uniform(-0.01, 0.01)
    T, cells, bins, v_max, n = case["T"], case["cells"], case["bins"], case["v_max"], case["packets"]
    if case["clouds"] > 1:
        tau0 *= 10.0 ** (0.5 * scale)
        T *= 10.0 ** (-0.5 * scale)
        cells, bins = max(4, int(cells * (1.0 + 0.3 * scale))), max(8, int(bins * (1.0 - 0.2 * scale)))
        v_max *= 1.0 + 0.5 * scale
    if case["geometry"] == "sphere":
        u = v_max / (12.85 * math.sqrt(T / 1.0e4))
        x_max = 6.0 * (4.702e-4 * math.sqrt(1.0e4 / T) * tau0) ** (1.0 / 3.0) + 1.2 * u
        m = media.sphere(tau0, T, cells, max(bins, 1), x_max=max(x_max, 3.0), v_max=v_max, n_packets=n,
                         tau_threshold=case["tau_th"])
    else:
        x_max = 6.0 * (4.702e-4 * math.sqrt(1.0e4 / T) * tau0) ** (1.0 / 3.0)
        m = media.slab(tau0, T, cells, max(bins, 1), x_max=max(x_max, 3.0), n_packets=n,
                       tau_threshold=case["tau_th"])
    kw = {}
    if case["grid"] == "efficient":
        dz = (2.0 if case["geometry"] == "slab" else 1.0) / cells
        kw["bin_edges"] = media.efficient_edges(4.702e-4 * math.sqrt(1.0e4 / T), case["tau0"], dz)
    if case["groups"]:
        kw["flags"] = media.GROUP_MC
    if case["dust"] > 0.0:
        kw["dust_abs"], kw["dust_sca"] = np.full(cells, case["dust"]), np.full(cells, 0.5 * case["dust"])
        if case["weights"]:
            kw["flags"] = kw.get("flags", 0) | media.DUST_WEIGHT
    if case["census"]:
        kw["census"] = np.linspace(0.0, 4.0, case["census"] + 1)
    return m.replace(**kw)


def _media(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["geometry"] == "cube":
        per = max(1, case["packets"] // case["sources"])
        return [media.cube(case["n"], seed=seed, sigma_v=case["sigma_v"], n_bins=case["bins"],
                           dv_bin=25.0 * 256 / case["bins"], n_sources=case["sources"], packets_per_source=per)]
    n = case["clouds"]
    return [_medium(case, rng, 0.0 if n == 1 else 2.0 * i / (n - 1) - 1.0) for i in range(n)]


def _attach_clouds(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(case["clouds"]):
        tau0 = case["tau0"] * 10.0 ** rng.uniform(-0.01, 0.01)
        x_max = 6.0 * (4.702e-4 * math.sqrt(1.0e4 / case["T"]) * case["tau0"]) ** (1.0 / 3.0)
        bins = int(round(2.0 * x_max / case["dx"]))
        out.append(media.sphere(tau0, case["T"], case["cells"], bins, x_max=x_max, v_max=case["v_max"],
                                n_packets=4096))
    return out


# ---- one call -----------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        n = case["batch"]
        x = torch.zeros((n, 16), device="cuda")
        x[:, :8] = torch.randn((n, 8), device="cuda", generator=g)
        y = torch.randn((n, 3), device="cuda", generator=g)
        y[:, 0] = (y[:, 0] > 0).float()
        y[:, 2] = 1.0 + 0.5 * y[:, 2]
        net = rddmc.Mdn(max_batch=n, seed=seed)
        return {"kind": kind, "net": net, "theta": net.params[:net.n_params].clone(), "x": x, "y": y}
    if kind == "data":
        dom = surrogate.Domain(tau_min=1.0e4, tau_max=case["tau_max"], dx_min=0.5, dx_max=4.5)
        return {"kind": kind, "probes": surrogate.sample_probes(case["probes"], dom, seed=seed), "dom": dom,
                "per_probe": case["per_probe"], "seed": seed}
    if kind == "attach":
        return {"kind": kind, "problem": rddmc.Problem(_attach_clouds(case, seed)),
                "net": rddmc.Mdn(max_batch=case["max_batch"], seed=seed), "dom": surrogate.use_domain()}
    meds = _media(case, seed)
    return {"kind": kind, "seed": seed, "media": meds, "problem": None if kind == "job" else rddmc.Problem(meds)}


def _results(problem):
    out = []
    for r in problem.results():
        d = {"spectrum": r.spectrum, "time_hist": r.time_hist, "step_hist": r.step_hist,
             "counts": np.array([r.launched, r.escaped, r.capped, r.steps_total, r.steps_max, r.to_mc, r.to_ddmc,
                                 r.reflected, r.mc_steps, r.surrogate_calls, r.absorbed], dtype=np.int64),
             "means": np.array([r.steps_mean, r.t_mean, r.t_var, r.escaped_w, r.t_mean_w, r.t_var_w])}
        for k in ("pixels", "census_bin", "census_path", "census_accel", "spectrum_w", "spectrum_w2"):
            if getattr(r, k) is not None:
                d[k] = getattr(r, k)
        out.append(d)
    return out


def run(state):
    kind = state["kind"]
    if kind == "train":
        # one minibatch step from the same point: loss, gradient and updated parameters
        net = state["net"]
        n = net.n_params
        net.params[:n].copy_(state["theta"])
        net.params[n:3 * n].zero_()
        net.step = 0
        loss = net.train_step(state["x"], state["y"], 2.0e-3)
        return {"loss": loss, "theta": net.params[:n], "grad": net.params[3 * n:4 * n]}
    if kind == "data":
        d = surrogate.generate_mixed(state["probes"], state["per_probe"], state["dom"], seed=state["seed"],
                                     step_budget=2.0e4, max_steps=1 << 30)
        return {"x": d.x, "y": d.y, "steps": d.steps}
    if kind == "attach":
        att = surrogate.Attached(state["problem"], state["net"], state["dom"])
        n = int(att.n_states)
        return {"records": att.buffer[att.buffer.numel() - 512 * n:].view(torch.float32).reshape(n, 128)[:, :114]}
    if kind == "job":
        problem = rddmc.Problem(state["media"])
        problem.run(seed=state["seed"])
        return _results(problem)
    problem = state["problem"]
    problem.reset()
    if kind == "exit":
        problem.run(seed=state["seed"], surrogate=rddmc.ExitKernel(problem).buffer)
    else:
        problem.run(seed=state["seed"])
    return _results(problem)


# ---- what a call cannot do without -----------------------------------------------------------

_MACS = 16 * 256 + 256 * 256 + 256 * 256 + 256 * 128     # products of one network evaluation
_PARAMS = _MACS + 3 * 256 + 128


def _windows(meds):
    """Each cloud's surrogate window (i_lo, i_hi, j_lo, j_hi) and the number of its states."""
    ws = [surrogate.window(m, surrogate.use_domain()) for m in meds]
    return [(w, (w[1] - w[0] + 1) * (w[3] - w[2] + 1) if w[1] >= w[0] else 0) for w in ws]


def work(case):
    """Walks: a DDMC step or MC event is at least 32 operations (half a Philox block, the path
    length, the event, the address); a packet takes about tau0 / dx^2 frequency steps on a uniform
    grid and half the squared cell count in spatial ones (the efficient grid's core bin skips
    the first); the state records are read and the tallies written once.  Tables: about 500
    operations per state (four error and Dawson functions), the input read and 40 bytes written."""
    kind = case["kind"]
    if kind == "train":
        n = case["batch"]
        return {"bytes": 4.0 * (19 * n + 8 * _PARAMS), "flops": 6.0 * n * _MACS}
    if kind == "data":
        rows = case["probes"] * case["per_probe"]
        return {"bytes": 4.0 * 19 * rows, "flops": 32.0 * 2.0e3 * rows}
    if kind == "attach":
        n = max(1, sum(k for _, k in _windows(_attach_clouds(case, 0))))
        return {"bytes": 512.0 * n + 2.0 * _PARAMS, "flops": 2.0 * n * _MACS}
    if case["geometry"] == "cube":
        states = case["n"] ** 3 * case["bins"]
        steps = 1.0e3 * (case["n"] / 24.0) ** 1.7 * case["packets"]
        return {"bytes": 40.0 * states if kind == "job" else 16.0 * min(states, steps),
                "flops": 32.0 * steps + (500.0 * states if kind == "job" else 0.0)}
    meds = _media(case, 0)
    nbytes = flops = 0.0
    for m in meds:
        states = m.n_cells_total * m.n_bins
        dx = float(np.max(np.diff(m.bin_edges)))
        scat = 0.0 if case["grid"] == "efficient" or kind == "exit" else case["tau0"] / max(dx, 0.05) ** 2
        if case["tau_th"] > 0.0:
            scat = case["tau0"]
        steps = (scat + 0.4 * m.n_cells_total ** 2 + 10.0) * m.n_packets
        nbytes += 16.0 * states + 8.0 * states * 2 * case["census"] + 8.0 * 2 * (m.n_bins + 2)
        flops += 32.0 * steps
        if kind == "job":
            nbytes += 40.0 * states + (16.0 * m.n_bins ** 2 if case["groups"] else 0.0)
            flops += 500.0 * states
        if kind == "exit":
            nbytes += 24.0 * states * m.n_bins / 4
            flops += 40.0 * states * m.n_bins
    return {"bytes": nbytes, "flops": flops}


# ---- 64-bit values ------------------------------------------------------------------------------

_SHAPES = [(16, 256), (256,), (256, 256), (256,), (256, 256), (256,), (256, 128), (128,)]


def _forward64(theta, x):
    parts, o = [], 0
    for s in _SHAPES:
        k = int(np.prod(s))
        parts.append(theta[o:o + k].reshape(s))
        o += k
    h = x
    for layer in range(4):
        h = h @ parts[2 * layer] + parts[2 * layer + 1]
        if layer < 3:
            h = 0.5 * h * torch.erfc(-h / math.sqrt(2.0))
    return h


def _nll64(o, y):
    logit = torch.log_softmax(o[:, :16], dim=1)
    face = torch.log_softmax(o[:, 16:48].reshape(-1, 16, 2), dim=2)
    f = torch.gather(face, 2, y[:, 0].long().reshape(-1, 1, 1).expand(-1, 16, 1))[:, :, 0]
    s1, s2 = o[:, 64:80].clamp(-6.0, 4.0), o[:, 96:112].clamp(-6.0, 4.0)
    rho = 0.95 * torch.tanh(o[:, 112:128])
    z1, z2 = (y[:, 1:2] - o[:, 48:64]) * torch.exp(-s1), (y[:, 2:3] - o[:, 80:96]) * torch.exp(-s2)
    om = 1.0 - rho * rho
    q = (z1 * z1 - 2.0 * rho * z1 * z2 + z2 * z2) / om
    ll = logit + f - math.log(2.0 * math.pi) - s1 - s2 - 0.5 * torch.log(om) - 0.5 * q
    return -torch.logsumexp(ll, dim=1).mean()


def _features64(m, w):
    """The eight network inputs of every window state, and its scales S and w."""
    f, e = np.asarray(m.faces[0]), np.asarray(m.bin_edges)
    T = float(m.temp[0])
    a, vth = 4.702e-4 * math.sqrt(1.0e4 / T), 12.85 * math.sqrt(T / 1.0e4)
    i, j = np.meshgrid(np.arange(w[0], w[1] + 1), np.arange(w[2], w[3] + 1), indexing="ij")
    i, j = i.ravel(), j.ravel()
    lo, hi = f[i], f[i + 1]
    wd, v3 = hi - lo, (hi ** 3 - lo ** 3) / 3.0
    tau = m.k0[i] * wd
    # the comoving shift of eq. 20 across each face; the velocity's sign follows the face's normal
    s0 = -m.f_mu * (m.vel[i] - m.vel[i - 1]) / vth
    s1 = -m.f_mu * (m.vel[i + 1] - m.vel[i]) / vth
    x = np.zeros((len(i), 16))
    x[:, 0] = (np.log10(tau) - 6.0) / 1.5
    x[:, 1] = (math.log10(a) + 3.3) / 0.6
    x[:, 2] = 0.5 * (e[j] + e[j + 1]) / 3.0
    x[:, 3] = np.log10(e[j + 1] - e[j]) / 0.7
    x[:, 4], x[:, 5] = s0, s1
    x[:, 6], x[:, 7] = 4.0 * (lo * lo / v3 * wd - 1.0), 4.0 * (hi * hi / v3 * wd - 1.0)
    return x, np.cbrt(a * tau), wd


def exact(case, seed):
    if case["kind"] == "train":
        s = prepare(case, seed)
        theta = s["theta"].double().requires_grad_(True)
        loss = _nll64(_forward64(theta, s["x"].double()), s["y"].double())
        (g,) = torch.autograd.grad(loss, theta)
        # first Adam step from zero moments: m / (1 - b1) = g, v / (1 - b2) = g^2
        new = theta.detach() - 2.0e-3 * g / (g.abs() + 1.0e-8)
        return {"loss": loss.detach().reshape(1), "theta": new, "grad": g}
    if case["kind"] == "attach":
        meds = _attach_clouds(case, seed)
        parts = [_features64(m, w) for m, (w, k) in zip(meds, _windows(meds)) if k]
        if not parts:
            return None
        x, S, wd = (np.concatenate(v) for v in zip(*parts))
        net = rddmc.Mdn(max_batch=32, seed=seed)
        theta = net.params[:net.n_params].double()
        o = _forward64(theta, torch.tensor(x, device="cuda"))
        r = torch.zeros((len(x), 114), dtype=torch.float64, device="cuda")
        r[:, :16] = torch.cumsum(torch.softmax(o[:, :16], dim=1), dim=1)
        r[:, 16:32] = torch.sigmoid(o[:, 16:48:2] - o[:, 17:48:2])
        r[:, 32:48], r[:, 64:80] = o[:, 48:64], o[:, 80:96]
        r[:, 48:64], r[:, 80:96] = torch.exp(o[:, 64:80].clamp(-6.0, 4.0)), torch.exp(o[:, 96:112].clamp(-6.0, 4.0))
        r[:, 96:112] = 0.95 * torch.tanh(o[:, 112:128])
        r[:, 112], r[:, 113] = torch.tensor(S, device="cuda"), torch.tensor(wd, device="cuda")
        return {"records": r}
    return None
