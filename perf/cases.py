"""Timed cases of the library: what a program that uses it has it do, through the binding.

Three kinds of work:

* "step": a running simulation is advanced by some steps and its diagnostics are read, as a run that
  records the line every few steps does.  One line or many, from a few hundred cells (a step there is
  a handful of launches) to tens of millions of particles, by each RICS backend, eager or from graphs.
* "forward", "gradient": the surrogate network over a batch, inference and loss with gradient.
* "train": a short training run of the surrogate, sample pool to parameters.

Simulations keep a bounded particle count (a density limit, or a line that loses as much as it gains),
so that a state can be stepped on for as long as a program likes.
"""
import math

import numpy as np
import torch

from paper_2609_17661_amd import Pic1D, pic1d, workloads

NPARAM = 50563
LAYERS = ((128, 4), (128, 128), (128, 128), (128, 128), (3, 128))
BOX = ((0.0, 8.0), (0.0, 1.0), (-2.0, 3.0), (0.3, 1.0))     # log10 gamma, s/L, log10 b, kT/keV


def _line(name, rics, r_eq, cells, ppc, steps, **kw):
    """A case of one line: defaults of the hot line at a density limit."""
    case = dict(name=name, kind="step", lines=1, rics=rics, r_eq=r_eq, cells=cells, ppc=ppc, steps=steps, init="hot",
                gamma_max=1.0e4, n_max=3.0, conversion="immediate", emission="perpendicular", atmosphere=False,
                sort=5, graph=0, warm=20)
    case.update(kw)
    return case


def listed():
    return [
        # one step of a small line, its diagnostics after each: launches and latency
        _line("small line single steps", "table", 4.0, 512, 64, 1, gamma_max=1.0e3, n_max=12.0,
              conversion="curvature", atmosphere=True, sort=10, warm=40),
        # the same size as a batch job: many steps a call, replayed from graphs
        _line("small line graph", "table", 4.0, 512, 64, 100, gamma_max=1.0e3, n_max=12.0, conversion="curvature",
              atmosphere=True, sort=10, graph=100, warm=40),
        # an ordinary line of odd size by the closed forms, with angle-resolved emission
        _line("odd line closed forms", "exact", 4.0, 9973, 61, 20, emission="dipole", atmosphere=True,
              sort=10),
        # the field line of the headline run after it has heated (most of its 20,000 steps)
        _line("long line heated", "table", 30.0, 65536, 200, 50, init="cold", n_max=0.0, conversion="curvature",
              atmosphere=True, sort=50, warm=3000),
        # the hot cascade held at the density limit: events, pairs and annihilation in every cell
        _line("hot line at the limit", "table", 4.0, 65536, 200, 10, warm=60),
        # many uneven lines in one state
        dict(name="many lines graph", kind="step", lines=40, rics="table", steps=50, graph=50, sort=50, warm=50),
        # the cascade on several long lines with atmospheres and ions, towards the density limit
        dict(name="cascade lines", kind="cascade", lines=8, rics="table", cells=32768, ppc=84, steps=20, graph=0,
             sort=50, warm=150),
        # the surrogate network in the pusher
        _line("surrogate line", "mlp", 4.0, 16384, 100, 5, warm=10),
        # the network on its own: a query, a large ragged batch, a training batch, a training run
        dict(name="forward small", kind="forward", n=1000),
        dict(name="forward large", kind="forward", n=1000003),
        dict(name="gradient", kind="gradient", n=8192),
        dict(name="train", kind="train", pool=1 << 18, batch=8192, steps=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("small", "line", "line", "limit", "lines", "cascade", "surrogate", "forward", "gradient", "train"))
    if kind == "small":
        c = _line("", "table", 4.0, _log(rng, 200, 2000), rng.randint(16, 100), rng.choice((1, 10, 50)),
                  gamma_max=1.0e3, n_max=12.0, conversion="curvature", atmosphere=True, sort=rng.choice((5, 10, 25)),
                  graph=rng.choice((0, 50)), warm=40)
    elif kind == "line":
        c = _line("", rng.choice(("table", "exact", "off")), rng.choice((4.0, 10.0, 30.0)), _log(rng, 3000, 50000),
                  rng.randint(24, 200), rng.choice((5, 20, 50)), conversion=rng.choice(("immediate", "curvature")),
                  emission=rng.choice(("perpendicular", "isotropic", "dipole")), atmosphere=True,
                  sort=rng.choice((5, 10, 50)))
    elif kind == "limit":
        c = _line("", rng.choice(("table", "exact")), 4.0, _log(rng, 8000, 65536), rng.randint(100, 200), 10, warm=60,
                  sort=rng.choice((5, 10)))
    elif kind == "lines":
        c = dict(kind="step", lines=rng.randint(5, 40), rics="table", steps=50, graph=rng.choice((0, 50)), sort=50,
                 warm=rng.randint(20, 80))
    elif kind == "cascade":
        c = dict(kind="cascade", lines=rng.randint(2, 8), rics="table", cells=_log(rng, 4000, 32768),
                 ppc=rng.randint(60, 84), steps=20, graph=0, sort=rng.choice((25, 50)), warm=100)
    elif kind == "surrogate":
        c = _line("", "mlp", 4.0, _log(rng, 500, 16384), rng.randint(30, 100), 5, warm=10)
    elif kind == "forward":
        c = dict(kind="forward", n=_log(rng, 16, 1000000))
    elif kind == "gradient":
        c = dict(kind="gradient", n=_log(rng, 64, 32768))
    else:
        c = dict(kind="train", pool=1 << 18, batch=_log(rng, 512, 8192), steps=rng.randint(20, 100))
    c.pop("name", None)
    return c


def _config(case, seed):
    if case["kind"] == "cascade":
        cfg = workloads.cfg5(n_lines=case["lines"], seed=0, n_cells=case["cells"], ppc=case["ppc"])
    elif case["lines"] > 1:
        cfg = workloads.cfg3(n_lines=case["lines"], seed=0, headroom=1.5)
    else:
        n, ppc = case["cells"], case["ppc"]
        # pairs up to the density limit of all species, appended slots between sorts included;
        # without one (0) the capacities of the long line
        limit = max(case["n_max"], 3.0) * ppc * n
        cap = int(1.5 * limit) + 65536
        cap_atm = (2000 + 2 * n) * ppc + 65536 if case["atmosphere"] else 0
        cfg = dict(kT_keV=0.5, j_twist=0.5, ppc0=float(ppc), pairs=True, conversion=case["conversion"],
                   emission=case["emission"], atmosphere=case["atmosphere"], mass_ratio=100.0,
                   nmax_over_n0=case["n_max"], rics=case["rics"],
                   lines=[dict(r_eq=case["r_eq"], n_cells=n, ppc_init=ppc, init=case["init"],
                               init_gamma_max=case["gamma_max"], capacity=[cap, cap, cap_atm, cap_atm])])
    cfg["sort_interval"] = case["sort"]
    cfg["seed"] = seed
    return cfg


def _samples(rng, n):
    """Inputs of the network in its box, inside the Planck cutoff, and its targets from the closed forms."""
    v0 = math.sqrt(0.75)                                        # the line of R_max = 4
    grid = np.linspace(-v0, v0, 20001)
    P = grid * np.sqrt(1 + 3 * grid**2) + np.arcsinh(math.sqrt(3) * grid) / math.sqrt(3)
    xs, os, have = [], [], 0
    while have < n:
        m = int(1.7 * (n - have)) + 64
        x = np.stack([rng.uniform(lo, hi, m) for lo, hi in BOX], axis=1).astype(np.float32).astype(np.float64)
        gam, b, th = 10.0 ** x[:, 0], 10.0 ** x[:, 2], x[:, 3] / 510.99895
        c = np.interp(P[-1] * (1 - 2 * x[:, 1]), P, grid)
        mu, r = 2 * c / np.sqrt(1 + 3 * c * c), 4 * (1 - c * c)
        y = b / (th * (gam - np.sqrt(gam * gam - 1) * mu))
        base = 2.8179403262e-13 * 1e6 / (4 * 3.8615926796e-11**2)
        with np.errstate(over="ignore", divide="ignore", invalid="ignore"):
            em1 = np.expm1(np.minimum(y, 100.0))
            o = np.stack([np.log10(base * th**3 * y**3 / em1 / r**2), np.log10(base * th**2 * y**2 / em1 / (r**2 * gam)),
                          np.log10(gam * (1 - 1 / np.sqrt(1 + 2 * b)))], axis=1)
        ok = y <= 80
        xs.append(x[ok])
        os.append(o[ok])
        have += int(ok.sum())
    return np.concatenate(xs)[:n], np.concatenate(os)[:n]


def _normalised(x):
    lo, hi = np.array(BOX).T
    return (x - lo) * (2 / (hi - lo)) - 1


def _silu(z):
    return z / (1 + np.exp(-z))


def _network(rng):
    """Parameters and target normalisation of a network for the closed forms: random hidden layers (twice
    Glorot's bound) and an output layer fitted to samples."""
    w = [rng.uniform(-1, 1, s) * 2 * math.sqrt(6 / (s[0] + s[1])) for s in LAYERS[:4]]
    b = [rng.uniform(-0.2, 0.2, s[0]) for s in LAYERS[:4]]
    x, o = _samples(rng, 2048)
    mean, std = o.mean(axis=0), o.std(axis=0)
    a = _normalised(x)
    for wl, bl in zip(w, b):
        a = _silu(a @ wl.T + bl)
    A = np.concatenate([a, np.ones((len(a), 1))], axis=1)
    fit = np.linalg.solve(A.T @ A + np.eye(129), A.T @ ((o - mean) / std))
    w.append(fit[:128].T)
    b.append(fit[128])
    params = np.concatenate([np.concatenate([wl.ravel(), bl]) for wl, bl in zip(w, b)])
    return params.astype(np.float32), np.concatenate([mean, std]).astype(np.float32)


def prepare(case, seed):
    if case["kind"] in ("step", "cascade"):
        cfg = _config(case, seed)
        if case["rics"] == "mlp":
            cfg["mlp_params"], cfg["mlp_norm"] = _network(np.random.default_rng(seed))
        sim = Pic1D(cfg)
        sim.step(case["warm"])
        if case["graph"]:
            sim.set_graph(case["graph"])
        return dict(kind="step", sim=sim, steps=case["steps"])
    if case["kind"] == "train":
        return dict(kind="train", seed=seed, n_samples=case["pool"], batch=case["batch"], steps=case["steps"])
    rng = np.random.default_rng(seed)
    params, norm = _network(rng)
    x, o = _samples(rng, case["n"])
    st = dict(kind=case["kind"], params=torch.from_numpy(params).cuda(), x=torch.from_numpy(x.astype(np.float32)).cuda())
    if case["kind"] == "gradient":
        st["t"] = torch.from_numpy(((o - norm[:3]) / norm[3:]).astype(np.float32)).cuda()
    return st


def run(state):
    kind = state["kind"]
    if kind == "step":
        sim = state["sim"]
        sim.step(state["steps"])
        if sim.n_lines > 1:
            return [sim.get_field(line) for line in range(sim.n_lines)]
        m = sim.moments(0)
        out = {k: m[k] for k in ("n", "j", "E", "pair_rate", "v_circuit", "energy_kinetic", "energy_field", "count")}
        out["counters"] = {k: m["counters"][k] for k in ("events", "pairs_created", "photons_escaped", "absorbed",
                                                         "limited", "pushed", "annihilated", "atm_injected")}
        return out
    if kind == "forward":
        return pic1d.mlp_forward(state["params"], state["x"])
    if kind == "gradient":
        return pic1d.mlp_loss_grad(state["params"], state["x"], state["t"])
    r = pic1d.mlp_train(seed=state["seed"], n_samples=state["n_samples"], batch=state["batch"], steps=state["steps"],
                        n_loss=0)
    return r["params"], r["norm"]


def work(case):
    kind = case["kind"]
    if kind in ("step", "cascade"):
        # cell, offset and momentum of every particle read and written in every step
        if kind == "cascade":
            n, cells = 11.0 * 32.0 * case["lines"] * case["cells"] * 0.54, case["lines"] * case["cells"]
        elif case["lines"] > 1:
            lines = workloads.cfg3(n_lines=case["lines"], seed=0)["lines"]
            n, cells = sum(2 * ln["ppc_init"] * ln["n_cells"] for ln in lines), sum(ln["n_cells"] for ln in lines)
        else:
            cells = case["cells"]
            n = max(2.0, case["n_max"]) * case["ppc"] * cells
        flops = 2 * 100096 * n if case["rics"] == "mlp" else 0.0
        return dict(bytes=case["steps"] * (24.0 * n + 32.0 * cells), flops=case["steps"] * flops)
    if kind == "forward":
        return dict(bytes=28.0 * case["n"] + 4 * NPARAM, flops=100096.0 * case["n"])
    if kind == "gradient":
        return dict(bytes=28.0 * case["n"] + 8 * NPARAM, flops=3 * 100096.0 * case["n"])
    return dict(bytes=32.0 * case["pool"] + case["steps"] * (32.0 * case["batch"] + 24 * NPARAM),
                flops=case["steps"] * 3 * 100096.0 * case["batch"])


def exact(case, seed):
    """The network's outputs and gradients in float64, on the bfloat16 weights that it is defined with.
    A simulation draws its events and takes its branches on float32 momenta: it has no such value."""
    if case["kind"] not in ("forward", "gradient"):
        return None
    st = prepare(case, seed)
    p = st["params"].double()
    w, b, k = [], [], 0
    for o, i in LAYERS:
        w.append(st["params"][k:k + o * i].bfloat16().double().reshape(o, i).requires_grad_())
        b.append(p[k + o * i:k + o * i + o].clone().requires_grad_())
        k += o * i + o
    lo = torch.tensor([v[0] for v in BOX], dtype=torch.float64, device=p.device)
    hi = torch.tensor([v[1] for v in BOX], dtype=torch.float64, device=p.device)

    def net(x):
        a = (x.double() - lo) * (2 / (hi - lo)) - 1
        for wl, bl in zip(w[:4], b[:4]):
            a = torch.nn.functional.silu(torch.nn.functional.linear(a, wl, bl))
        return torch.nn.functional.linear(a, w[4], b[4])

    if case["kind"] == "forward":
        with torch.no_grad():
            return torch.cat([net(x) for x in st["x"].split(1 << 16)])
    loss = (net(st["x"]) - st["t"].double()).square().mean()
    grads = torch.autograd.grad(loss, [v for pair in zip(w, b) for v in pair])
    return loss.item(), torch.cat([g.reshape(-1) for g in grads])
