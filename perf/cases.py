"""Performance cases of the library: the calls a program that packs circles makes.

A case is a dict of plain values.  ``listed()`` names the workloads that are
timed by name, ``draw(rng)`` gives one more of the same ranges; ``prepare``
makes what a program holds before the call (inputs from the seed, buffers and
workspaces it keeps), ``run`` makes ONE pass through the public entry points
and returns its outputs, ``work`` counts the bytes and operations the pass
cannot do without, and ``exact`` gives the outputs in 64 bits by plain torch
where they are computed numbers (a descent to convergence has none: its path
depends on every rounding).

Shapes: n circles of radius 1 in a container of radius R = sqrt(n / density),
densities around 0.84 as in the paper's instances (n = 300 .. 1000), and the
small n a first user tries.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2303_02650_amd as P

DEV = "cuda"
CUTOFF = 2.3


def listed():
    return [
        # the smallest call: one start, descended to convergence by a program
        # that must not allocate (a serving loop); latency of one instance
        {"name": "descend_1x20", "kind": "descend", "B": 1, "n_lo": 20, "n_hi": 20,
         "density": 0.74, "noalloc": True},
        # the headline: 256 random starts of n = 1000 to convergence
        {"name": "descend_256x1000", "kind": "descend", "B": 256, "n_lo": 1000, "n_hi": 1000,
         "density": 0.8353, "noalloc": False},
        # one iteration of SED over 128 chains of mixed size: plan, perturb,
        # descend the candidates (several hundred), verify, select
        {"name": "sed_128x300_1000", "kind": "sed", "B": 128, "n_lo": 300, "n_hi": 1000,
         "density": 0.84},
        # the container adjustment that ends every round of the framework
        {"name": "adjust_64x1000", "kind": "adjust", "B": 64, "n": 1000, "density": 0.8353},
        # geometric batch descent (Alg. 1 over a block grid), a fixed budget
        {"name": "gbo_64x1000", "kind": "gbo", "B": 64, "n": 1000, "density": 0.845,
         "blocks": 4, "max_iter": 300},
        # Alg. 1 over the paper's five sector batches, a fixed budget
        {"name": "kbatch5_128x1000", "kind": "kbatch", "B": 128, "n": 1000, "density": 0.845,
         "k": 5, "partition": "sector", "max_iter": 200},
        # the paper's dense inverse-Hessian matrices, one batch, a fixed budget
        {"name": "dense1_64x1000", "kind": "dense", "B": 64, "n": 1000, "density": 0.845,
         "k": 1, "max_iter": 100},
        # energies of new layouts: neighbor lists built, then energy and gradient
        {"name": "evaluate_4096x1000", "kind": "evaluate", "B": 4096, "n": 1000,
         "density": 0.8353, "form": 2},
        # energy and gradient over kept lists, the largest batch
        {"name": "sweep_65536x1000", "kind": "sweep", "B": 65536, "n": 1000, "density": 0.8353,
         "form": 2},
        # FP64 check of finished layouts
        {"name": "verify_2048x1000", "kind": "verify", "B": 2048, "n": 1000, "density": 0.8353},
        # the learned proposal's scoring: features and network of 4096
        # candidate relocations per instance
        {"name": "score_128x4096", "kind": "score", "B": 128, "n": 1000, "density": 0.845,
         "cands": 4096},
        # one Adam step of the proposal network on a minibatch
        {"name": "train_8192", "kind": "train", "rows": 8192},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["descend", "descend", "sed", "adjust", "gbo", "kbatch", "dense", "evaluate",
                       "evaluate", "sweep", "verify", "score", "train"])
    dens = round(rng.uniform(0.80, 0.85), 4)
    if kind == "descend":
        lo = _log_int(rng, 20, 1000)
        hi = lo if rng.random() < 0.5 else rng.randint(lo, min(1000, 3 * lo))
        return {"kind": kind, "B": _log_int(rng, 1, 256), "n_lo": lo, "n_hi": hi, "density": dens,
                "noalloc": rng.random() < 0.5}
    if kind == "sed":
        lo = rng.randint(100, 600)
        return {"kind": kind, "B": _log_int(rng, 4, 128), "n_lo": lo,
                "n_hi": rng.randint(lo, 1000), "density": dens}
    if kind == "adjust":
        return {"kind": kind, "B": _log_int(rng, 1, 64), "n": _log_int(rng, 20, 1000),
                "density": dens}
    if kind == "gbo":
        return {"kind": kind, "B": _log_int(rng, 4, 64), "n": rng.randint(300, 1000),
                "density": dens, "blocks": rng.randint(4, 6), "max_iter": rng.randint(50, 300)}
    if kind == "kbatch":
        return {"kind": kind, "B": _log_int(rng, 4, 128), "n": rng.randint(300, 1000),
                "density": dens, "k": rng.randint(1, 7),
                "partition": rng.choice(["sector", "annulus", "fence"]),
                "max_iter": rng.randint(30, 120)}
    if kind == "dense":
        return {"kind": kind, "B": _log_int(rng, 4, 64), "n": rng.randint(300, 1000),
                "density": dens, "k": rng.randint(1, 6), "max_iter": rng.randint(20, 80)}
    if kind == "evaluate":
        return {"kind": kind, "B": _log_int(rng, 1, 4096), "n": _log_int(rng, 20, 1000),
                "density": dens, "form": rng.randint(0, 2)}
    if kind == "sweep":
        return {"kind": kind, "B": _log_int(rng, 16, 65536), "n": rng.randint(100, 1000),
                "density": dens, "form": rng.randint(0, 2)}
    if kind == "verify":
        return {"kind": kind, "B": _log_int(rng, 1, 2048), "n": _log_int(rng, 20, 1000),
                "density": dens}
    if kind == "score":
        return {"kind": kind, "B": _log_int(rng, 4, 128), "n": rng.randint(100, 1000),
                "density": dens, "cands": _log_int(rng, 64, 4096)}
    return {"kind": kind, "rows": _log_int(rng, 50, 8192)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _sizes(case):
    """Instance sizes (those of a mixed batch belong to the case, not to the
    seed) and radii on the host."""
    B = case["B"]
    if "n" in case:
        n = np.full(B, case["n"], dtype=np.int64)
    else:
        n = np.random.default_rng(B).integers(case["n_lo"], case["n_hi"] + 1, size=B)
    return n, np.sqrt(n / case["density"])


def _instances(n, R):
    offset = np.zeros(len(n) + 1, dtype=np.int32)
    offset[1:] = np.cumsum(n)
    return P.DeviceInstances.from_host(offset, R, device=DEV)


def _disk(n, R, seed):
    """Centres uniform in the disk of radius R - 1 (the random starts)."""
    total = int(n.sum())
    u = torch.rand(total, 2, device=DEV, generator=_gen(seed))
    Rt = torch.from_numpy(R.astype(np.float32)).to(DEV).repeat_interleave(
        torch.from_numpy(n).to(DEV))
    r, th = (Rt - 1.0) * u[:, 0].sqrt(), 2.0 * math.pi * u[:, 1]
    return torch.stack([r * th.cos(), r * th.sin()], dim=1).reshape(-1)


def _hex(n, R):
    """The n points of a hexagonal lattice nearest the centre, scaled to fill
    the disk of radius R - 1: close to what a descent ends on."""
    m = int(math.sqrt(n)) + 3
    i, j = np.meshgrid(np.arange(-m, m + 1), np.arange(-m, m + 1))
    p = np.stack([(i + 0.5 * (j & 1)).ravel() + 0.1, (j * math.sqrt(3.0) / 2.0).ravel() + 0.05], axis=1)
    p = p[np.argsort((p * p).sum(1), kind="stable")[:n]]
    return p * ((R - 1.0) / max(1e-9, float(np.sqrt((p * p).sum(1)).max())))


def _packed(n, R, seed, jitter):
    """Nearly packed layouts: the lattice of every instance, turned by an
    angle of its own and shaken."""
    made = {}
    for a, r in zip(n, R):
        if int(a) not in made:
            made[int(a)] = torch.from_numpy(_hex(int(a), float(r)).astype(np.float32)).to(DEV)
    if len(made) == 1:
        base = next(iter(made.values())).repeat(len(n), 1)
    else:
        base = torch.cat([made[int(a)] for a in n])
    g = _gen(seed)
    th = (2.0 * math.pi) * torch.rand(len(n), device=DEV, generator=g)
    th = th.repeat_interleave(torch.from_numpy(n).to(DEV))
    c, s = th.cos(), th.sin()
    xy = torch.stack([c * base[:, 0] - s * base[:, 1], s * base[:, 0] + c * base[:, 1]], dim=1)
    return (xy + jitter * torch.randn(xy.shape, device=DEV, generator=g)).reshape(-1)


def _params(max_iter=5000):
    return P.DescentParams(max_iter=max_iter, g_tol=1e-6, ftol=1e-7, ftol_window=20,
                           contact_margin=1e-4)


def _bytes(count):
    return torch.empty(max(1, count), dtype=torch.uint8, device=DEV)


def _result(out):
    """The fields of a result buffer (views, nothing is copied)."""
    r = out.view(-1, P.RESULT_DTYPE.itemsize)
    return {"counts": r[:, 0:16].view(torch.int32), "pairs": r[:, 16:24].view(torch.int64),
            "E32_gnorm": r[:, 24:32].view(torch.float32), "E64": r[:, 32:40].view(torch.float64),
            "cell_evals": r[:, 40:44].view(torch.int32)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _prepare_train(case, seed)
    n, R = _sizes(case)
    inst = _instances(n, R)
    s = {"case": case, "inst": inst}
    B = inst.B
    if kind in ("descend", "gbo", "kbatch", "dense", "adjust"):
        s["xy0"] = _packed(n, R, seed, 0.05) if kind == "adjust" else _disk(n, R, seed)
        s["xy"] = s["xy0"].clone()
        s["out"] = _bytes(B * P.RESULT_DTYPE.itemsize)
        s["p"] = _params(case.get("max_iter", 5000)).c()
    if kind == "descend" and not case["noalloc"]:
        s["ws"] = _bytes(P.pecc_lbfgs_descend_workspace_size(inst))
    elif kind == "adjust":
        s["ws"] = _bytes(P.pecc_adjust_container_workspace_size(inst))
        s["R_out"] = torch.empty(B, dtype=torch.float32, device=DEV)
    elif kind == "gbo":
        s["ws"] = _bytes(P.pecc_gbo_descend_workspace_size(inst, case["blocks"]))
    elif kind == "kbatch":
        s["part"] = P.partition(inst, s["xy0"], case["partition"], case["k"])
        s["ws"] = _bytes(P.pecc_gbo_kbatch_descend_workspace_size(inst))
    elif kind == "dense":
        s["part"] = P.partition(inst, s["xy0"], "sector", case["k"])
        s["max_batch"] = -(-case["n"] // case["k"])
        s["ws"] = _bytes(P.pecc_gbo_kbatch_bfgs_workspace_size(inst, s["max_batch"]))
    elif kind == "sed":
        _prepare_sed(s, n, R, seed)
    elif kind in ("evaluate", "sweep"):
        s["xy"] = _disk(n, R, seed)
        s["E"] = torch.empty(B, dtype=torch.float32, device=DEV)
        s["g"] = torch.empty_like(s["xy"])
        if kind == "sweep":
            s["row"], s["col"] = P.build_neighbors(inst, s["xy"], CUTOFF, 0.0, case["form"])
            s["col"] = s["col"].clone()
        else:
            s["cap"] = 8 * inst.total_n
            s["row"] = torch.empty(inst.total_n + 1, dtype=torch.int32, device=DEV)
            s["col"] = torch.zeros(s["cap"], dtype=torch.int16 if case["form"] == P.LIST_LOCAL16
                                   else torch.int32, device=DEV)
            s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
            s["ws"] = _bytes(P.pecc_build_neighbors_workspace_size(inst))
    elif kind == "verify":
        s["xy"] = _packed(n, R, seed, 0.01)
        s["e"], s["mp"], s["mc"] = (torch.empty(B, dtype=torch.float64, device=DEV) for _ in range(3))
        s["f"] = torch.empty(B, dtype=torch.int32, device=DEV)
    elif kind == "score":
        C = case["cands"]
        s["xy"] = _packed(n, R, seed, 0.05)
        g = _gen(seed + 1)
        s["cc"] = torch.randint(0, case["n"], (B * C,), device=DEV, generator=g, dtype=torch.int32)
        s["cd"] = _disk(np.full(B, C), R, seed + 2)
        s["w"] = _net(seed)
        s["feat"] = torch.empty(B * C, P.PECC_FEATURES, dtype=torch.float32, device=DEV)
        s["z"] = torch.empty(B * C, dtype=torch.float32, device=DEV)
    return s


def _prepare_sed(s, n, R, seed):
    """Chains between two iterations: layouts, energies 1e-6 .. 1 (the number
    of candidates follows from them), and the candidate buffers."""
    B, M = len(n), 25
    g = _gen(seed + 1)
    s["M"], s["p"], s["seed"] = M, _params().c(), seed
    s["xy0"] = _packed(n, R, seed, 0.05)
    s["E0"] = 10.0 ** (-6.0 * torch.rand(B, device=DEV, generator=g, dtype=torch.float64))
    s["xy"], s["xy_best"] = s["xy0"].clone(), s["xy0"].clone()
    s["E"], s["E_best"] = s["E0"].clone(), s["E0"].clone()
    s["m"] = torch.zeros(B, dtype=torch.int32, device=DEV)
    s["chosen"] = torch.zeros(B, dtype=torch.int32, device=DEV)
    S = B * M
    s["cand"] = P.DeviceInstances(
        offset=torch.zeros(S + 1, dtype=torch.int32, device=DEV),
        R=torch.zeros(S, dtype=torch.float32, device=DEV),
        R64=torch.zeros(S, dtype=torch.float64, device=DEV), max_n=s["inst"].max_n,
        total_n=M * s["inst"].total_n)
    s["cand_xy"] = torch.zeros(2 * s["cand"].total_n, dtype=torch.float32, device=DEV)
    s["cand_E"] = torch.zeros(S, dtype=torch.float64, device=DEV)
    s["out"] = _bytes(S * P.RESULT_DTYPE.itemsize)
    s["ws"] = _bytes(P.pecc_lbfgs_descend_workspace_size(s["cand"]))


def _net(seed):
    return P.init_params(seed, device=DEV)


def _prepare_train(case, seed):
    """A trainer in the middle of training (moments and step count set) and a
    minibatch of candidates' features with labels."""
    rows = case["rows"]
    g = _gen(seed)
    t = P.MlpTrainer(_net(seed), lr=2e-3, max_rows=rows)
    t.m.copy_(1e-3 * torch.randn(t.m.shape, device=DEV, generator=g))
    t.v.copy_(1e-6 + 1e-5 * torch.rand(t.v.shape, device=DEV, generator=g))
    t.step.fill_(200)
    f = torch.rand(rows, P.PECC_FEATURES, device=DEV, generator=g)
    y = (torch.rand(rows, device=DEV, generator=g) < 0.3).to(torch.float32)
    return {"case": case, "t": t, "f": f, "y": y}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "train":
        t = s["t"]
        loss = t.train_step(s["f"], s["y"])
        return {"loss": loss, "grad": t.grad, "params": t.params, "m": t.m, "v": t.v,
                "step": t.step}
    inst = s["inst"]
    if kind in ("descend", "gbo", "kbatch", "dense", "adjust"):
        s["xy"].copy_(s["xy0"])
        if kind == "descend":
            if case["noalloc"]:
                P.pecc_lbfgs_descend_noalloc(inst, s["xy"], s["p"], s["out"])
            else:
                P.pecc_lbfgs_descend(inst, s["xy"], s["p"], s["out"], s["ws"])
        elif kind == "gbo":
            P.pecc_gbo_descend(inst, s["xy"], s["p"], case["blocks"], 0, s["out"], s["ws"])
        elif kind == "kbatch":
            P.pecc_gbo_kbatch_descend(inst, s["xy"], s["part"], case["k"], 0, s["p"], s["out"],
                                      s["ws"])
        elif kind == "dense":
            P.pecc_gbo_kbatch_bfgs_descend(inst, s["xy"], s["part"], case["k"], 0, s["max_batch"],
                                           s["p"], s["out"], s["ws"])
        else:
            P.pecc_adjust_container(inst, s["xy"], s["p"], 1e-4, 35, s["R_out"], s["out"], s["ws"])
            return {"xy": s["xy"], "R": s["R_out"], **_result(s["out"])}
        return {"xy": s["xy"], **_result(s["out"])}
    if kind == "sed":
        for a, b in (("xy", "xy0"), ("xy_best", "xy0"), ("E", "E0"), ("E_best", "E0")):
            s[a].copy_(s[b])
        c = s["cand"]
        P.pecc_sed_plan(inst, s["E"], s["E_best"], s["M"], 1e-25, s["m"], c.offset, c.R, c.R64)
        P.pecc_sed_perturb(inst, s["xy"], s["M"], s["m"], c.offset, s["seed"], 0, s["cand_xy"])
        P.pecc_lbfgs_descend(c, s["cand_xy"], s["p"], s["out"], s["ws"])
        P.pecc_verify(c, s["cand_xy"], 1e-20, s["cand_E"], None, None, None)
        P.pecc_sed_select(inst, s["M"], s["m"], c.offset, s["cand_xy"], s["cand_E"], s["seed"], 0,
                          s["xy"], s["E"], s["xy_best"], s["E_best"], s["chosen"])
        return {"xy": s["xy"], "E": s["E"], "xy_best": s["xy_best"], "E_best": s["E_best"],
                "chosen": s["chosen"], "m": s["m"], "cand_E": s["cand_E"],
                "cand_offset": c.offset, "cand_xy": s["cand_xy"]}
    if kind == "evaluate":
        P.pecc_build_neighbors(inst, s["xy"], CUTOFF, 0.0, case["form"], s["row"], s["col"],
                               s["cap"], s["count"], s["ws"])
        P.pecc_energy_grad(inst, s["xy"], s["row"], s["col"], s["cap"], case["form"], 1.0, s["E"],
                           s["g"])
        return {"E": s["E"], "g": s["g"], "row": s["row"], "col": s["col"], "count": s["count"]}
    if kind == "sweep":
        P.pecc_energy_grad(inst, s["xy"], s["row"], s["col"], s["col"].numel(), case["form"], 1.0,
                           s["E"], s["g"])
        return {"E": s["E"], "g": s["g"]}
    if kind == "verify":
        P.pecc_verify(inst, s["xy"], 1e-20, s["e"], s["mp"], s["mc"], s["f"])
        return {"E": s["e"], "max_pair": s["mp"], "max_cont": s["mc"], "feasible": s["f"]}
    P.pecc_features(inst, s["xy"], case["cands"], s["cc"], s["cd"], s["feat"])
    P.pecc_mlp_forward(s["w"], s["feat"], s["feat"].shape[0], s["z"])
    return {"features": s["feat"], "logits": s["z"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _pairs(n, density):
    """Pairs closer than the list cutoff in a random layout (edges left out)."""
    R = math.sqrt(n / density)
    return 0.5 * n * n * (CUTOFF / max(R - 1.0, CUTOFF)) ** 2


def _eval_flops(n, density):
    """One evaluation and one iteration of the limited-memory update."""
    return 10 * _pairs(n, density) + 18 * n + 160 * n


def work(case):
    kind = case["kind"]
    if kind == "train":
        r = case["rows"]
        return {"bytes": 36 * r + 4 * 4801 * 7, "flops": 3 * 9344 * r}
    B, d = case["B"], case["density"]
    n = case["n"] if "n" in case else 0.5 * (case["n_lo"] + case["n_hi"])
    iters = 60 + 0.9 * n                  # a descent of a random start, about
    if kind == "descend":
        return {"bytes": B * (16 * n + 48), "flops": B * iters * _eval_flops(n, d)}
    if kind == "sed":
        c = 3.5 * B                       # candidates: J uniform in 1 .. 6
        return {"bytes": B * 24 * n + c * (16 * n + 48),
                "flops": c * iters * _eval_flops(n, d)}
    if kind == "adjust":
        return {"bytes": B * (16 * n + 56), "flops": B * 2 * iters * _eval_flops(n, d)}
    if kind == "gbo":
        return {"bytes": B * (16 * n + 48), "flops": B * case["max_iter"] * 2 * _eval_flops(n, d)}
    if kind == "kbatch":
        return {"bytes": B * (20 * n + 48), "flops": B * case["max_iter"] * 2 * _eval_flops(n, d)}
    if kind == "dense":
        size = (2.0 * n / case["k"]) ** 2 * case["k"]
        return {"bytes": B * case["max_iter"] * 8 * size,
                "flops": B * case["max_iter"] * 11 * size}
    p = _pairs(n, d)
    lists = (8 if case.get("form") == P.LIST_FULL else 4) * p
    if kind == "evaluate":
        return {"bytes": B * (16 * n + 4 * (n + 1) + lists + 4), "flops": B * 30 * p}
    if kind == "sweep":
        return {"bytes": B * (16 * n + 4 * (n + 1) + lists + 4), "flops": B * 20 * p}
    if kind == "verify":
        return {"bytes": B * (8 * n + 28), "flops": B * 8 * p}
    C = case["cands"]
    return {"bytes": B * (8 * n + C * 48) + 4 * 4801, "flops": B * C * (9344 + 2 * 5 * 15)}


# ---------------------------------------------------------------------------
# The outputs in 64 bits
# ---------------------------------------------------------------------------
def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(_prepare_train(case, seed))
    if kind not in ("evaluate", "sweep", "verify", "score"):
        return None
    n, R = _sizes(case)
    if kind == "score":
        return _exact_score(case, n, R, seed)
    xy = _packed(n, R, seed, 0.01) if kind == "verify" else _disk(n, R, seed)
    B, k = case["B"], case["n"]
    x = xy.view(B, k, 2).double()
    Rb = torch.from_numpy(R).to(DEV)
    if kind != "verify":
        Rb = Rb.float().double()
    E = torch.empty(B, dtype=torch.float64, device=DEV)
    mp, mc = torch.empty_like(E), torch.empty_like(E)
    grad = torch.empty_like(x) if kind != "verify" else None
    step = max(1, int(5e7 / (k * k)))
    eye = torch.eye(k, dtype=torch.bool, device=DEV)
    for a in range(0, B, step):
        p = x[a:a + step]
        dx = p[:, :, None, 0] - p[:, None, :, 0]
        dy = p[:, :, None, 1] - p[:, None, :, 1]
        l = (dx * dx + dy * dy).sqrt_()
        d = (2.0 - l).clamp_(min=0.0).masked_fill_(eye, 0.0)
        rho = p.square().sum(2).sqrt()
        d0 = (rho + 1.0 - Rb[a:a + step, None]).clamp(min=0.0)
        E[a:a + step] = 0.5 * (d * d).sum((1, 2)) + (d0 * d0).sum(1)
        mp[a:a + step], mc[a:a + step] = d.amax((1, 2)), d0.amax(1)
        if grad is not None:
            k2 = d.mul_(-2.0).div_(l.clamp_(min=1e-300))
            c = 2.0 * d0 / rho.clamp(min=1e-300)
            grad[a:a + step, :, 0] = (k2 * dx).sum(2) + c * p[:, :, 0]
            grad[a:a + step, :, 1] = (k2 * dy).sum(2) + c * p[:, :, 1]
    if kind == "verify":
        return {"E": E, "max_pair": mp, "max_cont": mc, "feasible": None}
    out = {"E": E, "g": grad.reshape(-1)}
    if kind == "evaluate":
        out |= {"row": None, "col": None, "count": None}
    return out


def _split(w):
    """The network's weights in 64 bits, matrices at their BF16 roundings."""
    q = w.to(torch.bfloat16).double()
    w = w.double()
    return (q[:512].view(64, 8), w[512:576], q[576:4672].view(64, 64), w[4672:4736], q[4736:4800],
            w[4800])


def _logits(parts, f):
    W1, b1, W2, b2, W3, b3 = parts
    gelu = torch.nn.functional.gelu
    return gelu(gelu(f @ W1.t() + b1) @ W2.t() + b2) @ W3 + b3


def _exact_score(case, n, R, seed):
    B, k, C = case["B"], case["n"], case["cands"]
    x = _packed(n, R, seed, 0.05).view(B, k, 2).double()
    g = _gen(seed + 1)
    cc = torch.randint(0, k, (B * C,), device=DEV, generator=g, dtype=torch.int32).view(B, C).long()
    cd = _disk(np.full(B, C), R, seed + 2).view(B, C, 2).double()
    feat = torch.empty(B, C, 8, dtype=torch.float64, device=DEV)
    for b in range(B):
        Rb = float(R[b])
        for h, q in ((0, x[b][cc[b]]), (4, cd[b])):
            l2 = (q[:, None, 0] - x[b][None, :, 0]).square() + (q[:, None, 1] - x[b][None, :, 1]).square()
            l2.scatter_(1, cc[b][:, None], 1e9)      # the circle itself is lifted out
            rho = q.square().sum(1).sqrt()
            e = (2.0 - l2.sqrt()).clamp(min=0.0).square().sum(1) + (rho + 1.0 - Rb).clamp(min=0.0).square()
            feat[b, :, h] = torch.log10(e + 1e-20) / 20.0 + 1.0
            feat[b, :, h + 1] = (l2 < 5.29).sum(1)
            feat[b, :, h + 2] = (Rb - 1.0 - rho) / Rb
            feat[b, :, h + 3] = (l2 < 16.0).sum(1) / (16.0 * math.pi)
    feat = feat.view(B * C, 8)
    parts = _split(_net(seed))
    z = torch.cat([_logits(parts, f) for f in feat.split(65536)])
    return {"features": feat, "logits": z}


def _exact_train(s):
    t = s["t"]
    parts = [p.clone().requires_grad_() for p in _split(t.params)]
    loss = torch.nn.functional.binary_cross_entropy_with_logits(
        _logits(parts, s["f"].double()), s["y"].double())
    grad = torch.cat([p.reshape(-1) for p in torch.autograd.grad(loss, parts)])
    hp, k = t.hp, int(t.step.item()) + 1
    b1, b2 = float(hp.beta1), float(hp.beta2)
    m = b1 * t.m.double() + (1.0 - b1) * grad
    v = b2 * t.v.double() + (1.0 - b2) * grad * grad
    p = t.params.double() - float(hp.lr) * (m / (1.0 - b1 ** k)) / (
        (v / (1.0 - b2 ** k)).sqrt() + float(hp.eps))
    return {"loss": loss.detach().reshape(1), "grad": grad, "params": p, "m": m, "v": v,
            "step": None}
