"""The workloads this library is used for, with inputs made on the GPU from a seed.

A renderer that learns to guide its paths alternates three things, and every case is one
of them, called through the package's public functions:

  fit      weighted MAP EM of the cells' mixtures on a batch of path vertices, followed
           where a renderer goes on to guide with them by the conditioning table;
  tree     the pre-subdivision of a kD-tree and its refinement with the vertices, which
           come in the order the paths were traced (not grouped by cell);
  guide    conditioning, sampling and pdf of the fitted mixtures at shading points (one
           fused call), from a handful of points to a whole wavefront;
  mis      the same by the separate calls, as a renderer that also samples the BSDF needs
           them: condition once, sample, and the pdf of directions drawn elsewhere;
  product  sampling from the product with a BSDF model, and that product's pdf;
  grad     value and gradient of the penalised log-likelihood for gradient refinement.

Each op has small calls (latency and launches count), ordinary ones and large ones; odd
and ragged sizes; and the options and component counts the library's users set.
"""
import math
import random

import torch

from paper_2111_13094_amd import autograd, sdmm

DEV = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64
LOG2PI = math.log(2.0 * math.pi)


# --- the cases -------------------------------------------------------------------------

def listed():
    return [
        # the smallest update: one leaf with a few hundred vertices, one step
        {"name": "fit one leaf", "op": "fit", "cells": 1, "mean": 300, "K": 16, "iters": 1, "eta": 1.0,
         "accurate": False, "table": False},
        # one mixture fitted to convergence: 20 batch iterations on 16384 vertices
        {"name": "fit single x20", "op": "fit", "cells": 1, "mean": 16384, "K": 16, "iters": 20, "eta": 1.0,
         "accurate": False, "table": False},
        # a renderer's iteration: a batch over 4096 cells, then the table it guides with
        {"name": "fit 4096 cells", "op": "fit", "cells": 4096, "mean": 1017, "K": 16, "iters": 1, "eta": 0.1,
         "accurate": False, "table": True},
        # ragged cells, a component count that fills no power of two, the accurate update
        {"name": "fit ragged accurate", "op": "fit", "cells": 701, "mean": 500, "K": 12, "iters": 2, "eta": 1.0,
         "accurate": True, "table": False},
        # one huge mixture: 2^24 vertices, 32 components
        {"name": "fit huge", "op": "fit", "cells": 1, "mean": 1 << 24, "K": 32, "iters": 1, "eta": 1.0,
         "accurate": False, "table": False},
        # the tree of a small early iteration and of a full one
        {"name": "tree small", "op": "tree", "n": 60001, "depth": 1, "split": 2000, "max_leaves": 512, "K": 16,
         "grouped": False},
        {"name": "tree large", "op": "tree", "n": 16616003, "depth": 3, "split": 16000, "max_leaves": 4096, "K": 16,
         "grouped": False},
        # guiding: a few paths, and a wavefront of 2^22 shading points with 4 draws each
        {"name": "guide small", "op": "guide", "cells": 512, "K": 16, "nq": 100, "ns": 1, "sorted": False,
         "uniforms": True},
        {"name": "guide wavefront", "op": "guide", "cells": 16384, "K": 16, "nq": 1 << 22, "ns": 4, "sorted": True,
         "uniforms": False},
        # multiple importance sampling with the BSDF: separate calls, points in path order
        {"name": "mis", "op": "mis", "cells": 4096, "K": 16, "nq": 500009, "ns": 1, "nd": 1, "sorted": False,
         "uniforms": True},
        # product sampling over a wavefront, with the product's pdf at a BSDF direction
        {"name": "product", "op": "product", "cells": 16384, "K": 16, "Kb": 16, "models": 1, "nq": 1 << 21, "ns": 4,
         "nd": 1, "sorted": True, "uniforms": False},
        # one gradient of the penalised log-likelihood over the 4096-cell batch
        {"name": "grad 4096 cells", "op": "grad", "cells": 4096, "mean": 1017, "K": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["fit", "fit", "fit", "tree", "tree", "guide", "guide", "mis", "product", "grad"])
    K = rng.choice([5, 8, 12, 16, 16, 16, 24, 32])
    if op == "fit":
        cells = _log_int(rng, 1, 6000)
        total = _log_int(rng, 300, 4200000)
        return {"op": op, "cells": cells, "mean": min(max(32, total // cells), 1 << 21), "K": K,
                "iters": rng.choice([1, 1, 1, 2, 5]) if total < 400000 else 1, "eta": rng.choice([1.0, 1.0, 0.1]),
                "accurate": False, "table": rng.random() < 0.5} | (
                    {"accurate": True, "eta": 1.0} if rng.random() < 0.2 else {})
    if op == "tree":
        n = _log_int(rng, 10000, 16000000)
        return {"op": op, "n": n, "depth": rng.choice([1, 2, 3]), "split": max(500, _log_int(rng, n // 1200 + 1, n // 20)),
                "max_leaves": 4096, "K": rng.choice([8, 16]), "grouped": rng.random() < 0.3}
    if op in ("guide", "mis"):
        cells = _log_int(rng, 1, 16384)
        c = {"op": op, "cells": cells, "K": K, "nq": _log_int(rng, 50, 2000000), "ns": rng.choice([1, 1, 2, 3, 4, 8]),
             "sorted": rng.random() < 0.5, "uniforms": rng.random() < 0.5}
        if op == "mis":
            c["nd"] = rng.choice([1, 1, 2, 4])
            c["nq"] = min(c["nq"], 1000000)
        return c
    if op == "product":
        return {"op": op, "cells": _log_int(rng, 1, 16384), "K": rng.choice([8, 12, 16, 16]),
                "Kb": rng.choice([5, 8, 16, 16]), "models": rng.choice([1, 1, 7]), "nq": _log_int(rng, 50, 1500000),
                "ns": rng.choice([1, 2, 4, 5]), "nd": rng.choice([1, 2]), "sorted": rng.random() < 0.5,
                "uniforms": rng.random() < 0.5}
    return {"op": op, "cells": _log_int(rng, 1, 4096), "mean": _log_int(rng, 64, 1017), "K": min(K, 16)}


# --- inputs ----------------------------------------------------------------------------
# Path vertices come from six von Mises-Fisher lobes that point at emitters outside the
# unit cube (so direction and position are correlated), with heavy-tailed weights of which
# a tenth are zero (black vertices).

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed & 0x7FFFFFFF)
    return g


def _rand(g, *shape, dtype=F64):
    return torch.rand(*shape, generator=g, device=DEV, dtype=dtype)


def _randn(g, *shape, dtype=F64):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype)


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _lobes():
    """The scene's six emitters: direction from the cube's centre, distance, concentration
    and share (fixed: the scene stays, the seed draws its paths)."""
    r = random.Random(1234)
    dirs = []
    while len(dirs) < 6:
        v = [r.gauss(0, 1) for _ in range(3)]
        n = math.sqrt(sum(x * x for x in v))
        v = [x / n for x in v]
        if all(sum(a * b for a, b in zip(v, d)) <= math.cos(math.radians(45)) for d in dirs):
            dirs.append(v)
    dist = [r.uniform(1.5, 3.0) for _ in range(6)]
    kappa = [math.exp(r.uniform(math.log(5.0), math.log(200.0))) for _ in range(6)]
    share = [r.expovariate(1.0) + 0.1 for _ in range(6)]
    emit = [[0.5 + s * x for x in d] for d, s in zip(dirs, dist)]
    t = lambda v: torch.tensor(v, device=DEV, dtype=torch.float32)  # noqa: E731
    return t(emit), t(kappa), t(share) / sum(share)


def _directions(g, pos):
    """One direction per position (float32 [n, 3])."""
    emit, kappa, share = _lobes()
    n = pos.shape[0]
    j = torch.searchsorted(share.cumsum(0)[:-1].contiguous(), _rand(g, n, dtype=torch.float32))
    mu, kap = _unit(emit[j] - pos), kappa[j]
    u, phi = _rand(g, n, dtype=torch.float32), _rand(g, n, dtype=torch.float32) * (2 * math.pi)
    w = (1.0 + torch.log(u + (1.0 - u) * torch.exp(-2.0 * kap)) / kap).clamp(-1.0, 1.0)
    helper = torch.zeros_like(mu)
    helper[:, 0] = (mu[:, 0].abs() < 0.9).float()
    helper[:, 1] = 1.0 - helper[:, 0]
    t1 = _unit(helper - (helper * mu).sum(-1, keepdim=True) * mu)
    t2 = torch.linalg.cross(mu, t1)
    r = (1.0 - w * w).clamp_min(0.0).sqrt()
    return _unit(w[:, None] * mu + r[:, None] * (phi.cos()[:, None] * t1 + phi.sin()[:, None] * t2))


def _vertices(g, pos, sigma=1.5, black=0.1):
    n = pos.shape[0]
    smp = torch.empty(7, n, device=DEV, dtype=torch.float32)
    smp[0:3] = _directions(g, pos).T
    smp[3:6] = pos.T
    w = torch.exp(sigma * _randn(g, n, dtype=torch.float32))
    w[_rand(g, n, dtype=torch.float32) < black] = 0.0
    smp[6] = w
    return smp


def _boxes(cells):
    """A grid over the unit cube with at least `cells` boxes; the first `cells` are used."""
    side = 1
    while side ** 3 < cells:
        side += 1
    i = torch.arange(cells, device=DEV)
    lo = torch.stack([i // (side * side), (i // side) % side, i % side], 1).to(F64) / side
    return lo, torch.full((cells, 3), 1.0 / side, device=DEV, dtype=F64)


def _batch(g, cells, mean, sigma=1.5, black=0.1):
    """Ragged cells (lognormal counts about `mean`, a few of them nearly empty)."""
    if cells == 1:
        counts = torch.tensor([mean], device=DEV)
    else:
        z = _randn(g, cells)
        counts = (mean * torch.exp(z - 0.5)).round().clamp(8, 8 * mean).long()
    off = torch.zeros(cells + 1, device=DEV, dtype=torch.int64)
    off[1:] = counts.cumsum(0)
    lo, size = _boxes(cells)
    cell = torch.repeat_interleave(torch.arange(cells, device=DEV), counts)
    pos = (lo[cell] + _rand(g, cell.numel(), 3, dtype=torch.float32) * size[cell]).float()
    return off, _vertices(g, pos, sigma, black), 8 * mean if cells > 1 else mean


def _tri_index():
    return [(d, e) for d in range(5) for e in range(d + 1)]


def _pack(cov):
    return torch.stack([cov[..., d, e] for d, e in _tri_index()], -1)


def _unpack(p):
    cov = torch.zeros(*p.shape[:-1], 5, 5, device=p.device, dtype=p.dtype)
    for q, (d, e) in enumerate(_tri_index()):
        cov[..., d, e] = p[..., q]
        cov[..., e, d] = p[..., q]
    return cov


def _box_mixtures(lo, size, K):
    """The initial mixture of a box: eight cube-vertex directions crossed with positions
    along its longest sides, wide covariances, equal weights."""
    C = lo.shape[0]
    n_dir = min(8, K)
    n_pos = (K + n_dir - 1) // n_dir
    d = size.max(1).values
    order = torch.argsort(size, dim=1, descending=True, stable=True)
    rows = torch.arange(C, device=DEV)
    mu_pos = (lo + 0.5 * size)[:, None, :].repeat(1, K, 1)
    mu_dir = torch.empty(C, K, 3, device=DEV, dtype=F64)
    for k in range(K):
        s, v = divmod(k, n_dir)
        if n_pos == 2:
            mu_pos[rows, k, order[:, 0]] += (-1.0 if s == 0 else 1.0) * d / 4
        elif n_pos == 4:
            mu_pos[rows, k, order[:, 0]] += (-1.0 if s % 2 == 0 else 1.0) * d / 4
            mu_pos[rows, k, order[:, 1]] += (-1.0 if s // 2 == 0 else 1.0) * d / 4
        elif n_pos > 1:
            mu_pos[rows, k, order[:, 0]] += ((s + 0.5) / n_pos - 0.5) * d
        mu_dir[:, k] = torch.tensor([-1.0 if (v >> b) & 1 else 1.0 for b in (2, 1, 0)], device=DEV,
                                    dtype=F64) / math.sqrt(3.0)
    cov = torch.zeros(C, K, 5, 5, device=DEV, dtype=F64)
    cov[..., 0, 0] = cov[..., 1, 1] = 2 * math.pi / 8
    r = 2.0 * d / n_pos
    for a in range(2, 5):
        cov[..., a, a] = (r * r / 6.251388631170325)[:, None]
    return {"pi": torch.full((C * K,), 1.0 / K, device=DEV, dtype=F64), "mu_dir": mu_dir.reshape(-1).contiguous(),
            "mu_pos": mu_pos.reshape(-1).contiguous(), "cov": _pack(cov).reshape(-1).contiguous()}


def _fitted_mixtures(g, lo, size, K, dir_sd=(0.05, 0.4)):
    """Mixtures as a fit leaves them: components about the directions in which the
    emitters are seen from their positions, direction and position correlated, weights
    spread over two orders of magnitude."""
    C = lo.shape[0]
    n = C * K
    mu_pos = (lo[:, None] + (0.1 + 0.8 * _rand(g, C, K, 3)) * size[:, None]).reshape(n, 3)
    mu_dir = _unit(_directions(g, mu_pos.float()).to(F64))
    sd = torch.empty(n, 5, device=DEV, dtype=F64)
    sd[:, :2] = dir_sd[0] * (dir_sd[1] / dir_sd[0]) ** _rand(g, n, 1) * (0.7 + 0.6 * _rand(g, n, 2))
    sd[:, 2:] = (0.15 + 0.3 * _rand(g, n, 3)) * size.repeat_interleave(K, 0)
    low = 0.35 * _randn(g, n, 5, 5).tril(-1) + torch.eye(5, device=DEV, dtype=F64)
    low = sd[:, :, None] * low / low.norm(dim=2, keepdim=True)
    e = torch.exp(1.2 * _randn(g, C, K))
    return {"pi": (e / e.sum(1, keepdim=True)).reshape(-1), "mu_dir": mu_dir.reshape(-1).contiguous(),
            "mu_pos": mu_pos.reshape(-1).contiguous(), "cov": _pack(low @ low.mT).reshape(-1).contiguous()}


BSDF_LO, BSDF_HI = (0.0, 0.0, 0.05), (1.4, 2 * math.pi, 0.6)  # polar angle, azimuth, roughness


def _bsdf_models(g, n_models, Kb):
    n = n_models * Kb
    d = _randn(g, n, 3)
    d[:, 2] = d[:, 2].abs() + 0.6
    lo, hi = (torch.tensor(v, device=DEV, dtype=F64) for v in (BSDF_LO, BSDF_HI))
    sd = torch.empty(n, 5, device=DEV, dtype=F64)
    sd[:, :2] = (0.08 + 0.27 * _rand(g, n, 1)) * (0.8 + 0.4 * _rand(g, n, 2))
    sd[:, 2:] = torch.tensor([0.25, 0.8, 0.1], device=DEV, dtype=F64)
    low = 0.3 * (2 * _rand(g, n, 5, 5) - 1).tril(-1) + torch.eye(5, device=DEV, dtype=F64)
    low = sd[:, :, None] * low / low.norm(dim=2, keepdim=True)
    e = -torch.log(1 - _rand(g, n_models, Kb)) - torch.log(1 - _rand(g, n_models, Kb))
    return {"pi": (e / e.sum(1, keepdim=True)).reshape(-1), "mu_dir": _unit(d).reshape(-1).contiguous(),
            "mu_pos": (lo + _rand(g, n, 3) * (hi - lo)).reshape(-1).contiguous(),
            "cov": _pack(low @ low.mT).reshape(-1).contiguous()}


def _points(g, c, lo, size):
    cell = torch.randint(0, c["cells"], (c["nq"],), generator=g, device=DEV)
    if c["sorted"]:
        cell = cell.sort().values
    pos = (lo[cell] + _rand(g, c["nq"], 3) * size[cell]).float()
    return pos, cell.to(torch.int32)


def _rotations(g, n):
    q = _unit(_randn(g, n, 4))
    w, x, y, z = q.T
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                        2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                        2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]).float().contiguous()


def _inputs(case, seed):
    """Everything a case's program holds before it calls the library, as plain tensors."""
    g = _gen(seed)
    op = case["op"]
    if op == "fit":
        huge = case["mean"] > 1 << 20
        off, smp, bound = _batch(g, case["cells"], case["mean"], 2.5 if huge else 1.5, 0.0 if huge else 0.1)
        return {"off": off, "smp": smp, "bound": bound, "mix": _box_mixtures(*_boxes(case["cells"]), case["K"])}
    if op == "grad":
        off, smp, _ = _batch(g, case["cells"], case["mean"])
        return {"off": off, "smp": smp, "mix": _fitted_mixtures(g, *_boxes(case["cells"]), case["K"], (0.1, 0.6))}
    if op == "tree":
        n = case["n"]
        u = _rand(g, n, 3, dtype=torch.float32)
        pos = u * torch.sqrt(_rand(g, n, 1, dtype=torch.float32))  # denser towards a corner
        if case["grouped"]:
            side = (pos * 16).long()
            pos = pos[torch.argsort((side[:, 0] * 16 + side[:, 1]) * 16 + side[:, 2], stable=True)]
        return {"smp": _vertices(g, pos)}
    lo, size = _boxes(case["cells"])
    mix = _fitted_mixtures(g, lo, size, case["K"])
    pos, cell = _points(g, case, lo, size)
    out = {"mix": mix, "qpos": pos.T.contiguous(), "qcell": cell, "seed": (seed * 2654435761) & 0xFFFFFFFF,
           "u": _rand(g, 3, case["nq"] * case["ns"], dtype=torch.float32) if case["uniforms"] else None}
    if op in ("mis", "product"):  # directions a BSDF sampler drew at the same points
        out["dirs"] = _directions(g, pos.repeat_interleave(case["nd"], 0)).T.contiguous()
    if op == "product":
        l3, h3 = (torch.tensor(v, device=DEV, dtype=F64) for v in (BSDF_LO, BSDF_HI))
        out["bmix"] = _bsdf_models(g, case["models"], case["Kb"])
        out["bpar"] = (l3 + _rand(g, case["nq"], 3) * (h3 - l3)).float().T.contiguous()
        out["bcell"] = torch.randint(0, case["models"], (case["nq"],), generator=g, device=DEV).to(torch.int32)
        out["frames"] = _rotations(g, case["nq"])
    return out


# --- the program around the call, and the call -----------------------------------------

def prepare(case, seed):
    s = {"case": dict(case), **_inputs(case, seed)}
    op, K = case["op"], case["K"]
    if op == "fit":
        C, N = case["cells"], s["smp"].shape[1]
        s["state"] = sdmm.new_state(C, K, DEV)
        s["opts"] = sdmm.default_opts(K, iters=case["iters"], eta=case["eta"], max_cell_samples=s["bound"],
                                      flags=sdmm.FLAG_ACCURATE_SIGMA if case["accurate"] else 0)
        s["status"] = torch.empty(C, dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(sdmm.workspace_bytes(C, K, N, s["opts"]), dtype=torch.uint8, device=DEV)
        s["table"] = torch.empty(C * K * sdmm.COND_TABLE_STRIDE, device=DEV) if case["table"] else None
    elif op == "grad":
        C, N = case["cells"], s["smp"].shape[1]
        s["opts"] = sdmm.default_opts(K, prior_mode=sdmm.PRIOR_FIXED, prior_scale=1e-3)
        s["ws"] = torch.empty(sdmm.workspace_bytes(C, K, N, s["opts"]), dtype=torch.uint8, device=DEV)
        s["params"] = autograd.params_from_mixture(s["mix"], C, K)
    elif op == "tree":
        m = case["max_leaves"]
        z = lambda n: torch.zeros(n, device=DEV, dtype=F64)  # noqa: E731
        s["tree"] = sdmm.new_tree(m, DEV)
        s["mix"] = {"pi": z(m * K), "mu_dir": z(m * K * 3), "mu_pos": z(m * K * 3), "cov": z(m * K * 15)}
        s["state"] = sdmm.new_state(m, K, DEV)
        s["ws"] = torch.empty(int(sdmm.lib().sdmm_tree_workspace_size(case["n"], m)), dtype=torch.uint8, device=DEV)
    else:
        s["table"] = sdmm.condition_prepare(s["mix"], case["cells"], K)
        if op == "product":
            s["btable"] = sdmm.condition_prepare(s["bmix"], case["models"], case["Kb"])
    return s


def run(s):
    c = s["case"]
    op, K = c["op"], c["K"]
    if op == "fit":
        sdmm.fit_mixtures(s["off"], s["smp"], s["mix"], s["state"], s["opts"], s["status"], s["ws"])
        if c["table"]:
            sdmm.condition_prepare(s["mix"], c["cells"], K, table=s["table"])
        return {"status": s["status"], "mix": s["mix"], "state": s["state"], "table": s["table"]}
    if op == "grad":
        p = s["params"]
        F, status = autograd.penalised_log_likelihood(p, s["off"], s["smp"], s["opts"], s["ws"])
        grads = torch.autograd.grad(F.sum(), [p["alpha"], p["delta"], p["mu_pos"], p["L"]])
        return {"F": F, "status": status, "grads": list(grads)}
    if op == "tree":
        t = s["tree"]
        sdmm.tree_init(t, c["depth"], (0.0, 0.0, 0.0), (1.0, 1.0, 1.0))
        out, off, n_leaves, status = sdmm.tree_refine(t, s["smp"], c["split"], s["mix"], s["state"], K,
                                                      workspace=s["ws"])
        # the mixtures are held for max_leaves cells, so a fit of them takes the offsets of as
        # many: the cells past the last leaf are empty
        off = torch.nn.functional.pad(off, (0, c["max_leaves"] + 1 - off.numel()), value=c["n"])
        return {"sorted": out, "offsets": off, "leaves": n_leaves, "status": status,
                "tree": {k: t[k] for k in ("counts", "axis", "left", "leaf", "split", "leaf_node", "lo", "hi", "init")},
                "mix": s["mix"], "state": s["state"]}
    C = c["cells"]
    if op == "guide":
        d, p, v = sdmm.condition_sample_pdf(s["table"], C, K, s["qpos"], s["qcell"], c["ns"], uniforms=s["u"],
                                            seed=s["seed"])
        return {"dirs": d, "pdf": p, "valid": v}
    if op == "mis":
        cw, cm = sdmm.condition(s["table"], C, K, s["qpos"], s["qcell"])
        d, p, v, k = sdmm.sample(s["table"], C, K, s["qcell"], cw, cm, c["ns"], uniforms=s["u"], seed=s["seed"],
                                 with_comp=True)
        other = sdmm.pdf(s["table"], C, K, s["qcell"], cw, cm, s["dirs"], c["nd"])
        return {"weights": cw, "means": cm, "dirs": d, "pdf": p, "valid": v, "comp": k, "other": other}
    d, p, v, _ = sdmm.product_sample(s["table"], C, K, s["qpos"], s["qcell"], s["btable"], c["models"], c["Kb"],
                                     s["bpar"], s["bcell"], s["frames"], c["ns"], uniforms=s["u"], seed=s["seed"])
    other = sdmm.product_pdf(s["table"], C, K, s["qpos"], s["qcell"], s["btable"], c["models"], c["Kb"], s["bpar"],
                             s["bcell"], s["frames"], s["dirs"])
    return {"dirs": d, "pdf": p, "valid": v, "other": other}


def work(case):
    """Bytes: every input once and every output once. Flops: 140 per sample-component pair
    of an E-step pass, 31 + 56 + ... per conditioned and evaluated component (the counts
    bench.py states)."""
    op, K = case["op"], case["K"]
    if op in ("fit", "grad"):
        N, CK = case["cells"] * case["mean"], case["cells"] * K
        if op == "grad":
            return {"bytes": 28 * N + CK * 8 * (24 + 24 + 21), "flops": 140 * N * K}
        per = case["iters"] * (2 if case["accurate"] else 1)
        return {"bytes": 28 * N + 2 * CK * 8 * (22 + 16) + (CK * 128 if case["table"] else 0),
                "flops": 140 * N * K * per}
    if op == "tree":
        return {"bytes": 56 * case["n"], "flops": 12 * case["n"]}
    nq, nd = case["nq"], case["nq"] * case["ns"]
    tab = case["cells"] * K * 128
    if op == "guide":
        return {"bytes": 16 * nq + (29 if case["uniforms"] else 17) * nd + min(tab, nq * K * 128),
                "flops": nq * 31 * K + nd * (K + 38 + 56 * K)}
    if op == "mis":
        np_ = nq * case["nd"]
        return {"bytes": 16 * nq + 2 * 12 * nq * K + (33 if case["uniforms"] else 21) * nd + 16 * np_
                + min(tab, nq * K * 128), "flops": nq * 31 * K + nd * (K + 38 + 56 * K) + np_ * 56 * K}
    np_, Kb = nq * case["nd"], case["Kb"]
    return {"bytes": 68 * nq + (29 if case["uniforms"] else 17) * nd + 16 * np_ + min(tab, nq * K * 128),
            "flops": nq * (31 * K + 31 * Kb + 342 + 440 * K) + nd * (2 * K + 39 + 71 * K) + np_ * 71 * K}


# --- the same in 64 bits, in plain torch -----------------------------------------------

def _frame(mu):
    """Rows (t1, t2, mu) of the branchless basis about mu [..., 3] -> [..., 3, 3]."""
    x, y, z = mu.unbind(-1)
    sg = torch.copysign(torch.ones_like(z), z)
    a = -1.0 / (sg + z)
    b = x * y * a
    t1 = torch.stack([1.0 + sg * x * x * a, sg * b, -sg * x], -1)
    t2 = torch.stack([b, sg + y * y * a, -y], -1)
    return torch.stack([t1, t2, mu], -2)


def _log(R, w):
    """Tangent coordinates of directions w [..., 3] in frames R [..., 3, 3], with theta / sin theta."""
    v = (R * w.unsqueeze(-2)).sum(-1)
    s = torch.hypot(v[..., 0], v[..., 1]).clamp_min(1e-300)
    f = torch.atan2(s, v[..., 2]) / s
    f = torch.where(s > 1e-12, f, torch.ones_like(f))
    return f.unsqueeze(-1) * v[..., :2], f, v


def _exp(R, nu):
    r = torch.hypot(nu[..., 0], nu[..., 1])
    sc = torch.where(r > 1e-9, torch.sin(r) / r.clamp_min(1e-300), torch.ones_like(r))
    v = torch.cat([nu * sc.unsqueeze(-1), torch.cos(r).unsqueeze(-1)], -1)
    return (R * v.unsqueeze(-1)).sum(-2)


def _exp_jacobian(nu):
    """d (nu sinc r, cos r) / d nu [..., 3, 2]."""
    a, b = nu.unbind(-1)
    r2 = a * a + b * b
    r = r2.sqrt()
    small = r < 1e-2
    rs = torch.where(small, torch.ones_like(r), r)
    s = torch.where(small, 1 - r2 / 6 + r2 * r2 / 120, torch.sin(rs) / rs)
    c = torch.where(small, -1.0 / 3 + r2 / 30 - r2 * r2 / 840, (torch.cos(rs) - torch.sin(rs) / rs) / (rs * rs))
    return torch.stack([torch.stack([s + a * a * c, a * b * c], -1), torch.stack([a * b * c, s + b * b * c], -1),
                        torch.stack([-a * s, -b * s], -1)], -2)


def _mixture64(mix, C, K):
    return (mix["pi"].reshape(C, K), mix["mu_dir"].reshape(C, K, 3), mix["mu_pos"].reshape(C, K, 3),
            _unpack(mix["cov"].reshape(C, K, 15)))


def _log_density(R, mux, Li, logc, w, p):
    """log pi_k N5(y_k) and y_k of samples (w, p) [n, 3] under their components [n, K, ...]."""
    nu = _log(R, w[:, None])[0]
    y = torch.cat([nu, p[:, None] - mux], -1)
    z = (Li * y.unsqueeze(-2)).sum(-1)
    return logc - 0.5 * (z * z).sum(-1), y


def _stats(off, smp, pi, mud, mux, cov):
    """Sums over each cell's samples: W, M, S0 [C, K], S1 [C, K, 5], S2 [C, K, 15]."""
    C, K = pi.shape
    R = _frame(mud)
    L = torch.linalg.cholesky(cov)
    Li = torch.linalg.solve_triangular(L, torch.eye(5, device=DEV, dtype=F64).expand_as(L), upper=False)
    logc = pi.log() - L.diagonal(dim1=-2, dim2=-1).log().sum(-1) - 2.5 * LOG2PI
    N = smp.shape[1]
    cell = torch.repeat_interleave(torch.arange(C, device=DEV), off[1:] - off[:-1])
    S = torch.zeros(C, K, 21, device=DEV, dtype=F64)
    idx = _tri_index()
    step = max(1, (1 << 22) // K)
    for a in range(0, N, step):
        b = min(N, a + step)
        s, ce = smp[:, a:b].to(F64), cell[a:b]
        lo, hi = int(ce[0]), int(ce[-1]) + 1
        l, y = _log_density(R[ce], mux[ce], Li[ce], logc[ce], s[0:3].T, s[3:6].T)
        wr = s[6][:, None] * torch.softmax(l, -1)
        f = torch.stack([wr] + [wr * y[..., d] for d in range(5)] + [wr * y[..., d] * y[..., e] for d, e in idx], -1)
        if hi - lo == 1:
            S[lo] += f.sum(0)
        else:
            n = off[lo + 1:hi + 1].clamp(a, b) - off[lo:hi].clamp(a, b)
            S[lo:hi] += torch.segment_reduce(f.reshape(b - a, -1), "sum", lengths=n, axis=0,
                                             unsafe=True).reshape(hi - lo, K, 21)
        del f, l, y, wr
    w = smp[6].to(F64)
    cw = torch.zeros(C, device=DEV, dtype=F64).index_add_(0, cell, w)
    M = torch.zeros(C, device=DEV, dtype=F64).index_add_(0, cell, (w > 0).to(F64))
    return cw, M, S[..., 0], S[..., 1:6], _unpack(S[..., 6:])


def _exact_fit(case, x):
    C, K = case["cells"], case["K"]
    pi, mud, mux, cov = _mixture64(x["mix"], C, K)
    s0 = torch.zeros(C, K, device=DEV, dtype=F64)
    s2 = torch.zeros(C, K, 5, 5, device=DEV, dtype=F64)
    sw = torch.zeros(C, device=DEV, dtype=F64)
    q, a = 1.0 / K, 5.0 / K
    B = torch.diag(torch.tensor([0.1, 0.1, 1.0, 1.0, 1.0], device=DEV, dtype=F64) * a * 1e-4)
    for it in range(case["iters"]):
        eta = 1.0 if it == 0 else case["eta"]
        W, M, S0, S1, S2 = _stats(x["off"], x["smp"], pi, mud, mux, cov)
        ok = (M >= 16) & (W > 0)
        hW, hS0, hS1, hS2 = (1 - eta) * sw + eta * W, (1 - eta) * s0 + eta * S0, eta * S1, (1 - eta) * s2 + eta * S2
        beta = (eta / M.clamp_min(1.0))[:, None]
        Ws = torch.where(ok, hW, torch.ones_like(hW))[:, None]
        bar = hS0 / Ws
        live = ok[:, None] & (bar > 1e-12)
        d0 = torch.where(live, hS0, torch.ones_like(hS0))
        m = torch.where(live[..., None], hS1 / d0[..., None], torch.zeros_like(hS1))
        R = _frame(mud)
        new = _unit(_exp(R, m[..., :2]))
        J = _frame(new)[..., :2, :] @ (R.mT @ _exp_jacobian(m[..., :2]))
        T = torch.zeros(C, K, 5, 5, device=DEV, dtype=F64)
        T[..., :2, :2] = J
        T[..., 2:, 2:] = torch.eye(3, device=DEV, dtype=F64)
        TCT = T @ (hS2 - hS1[..., :, None] * hS1[..., None, :] / d0[..., None, None]) @ T.mT
        sig = (beta[..., None, None] * B + TCT / Ws[..., None, None]) / (beta * a + bar)[..., None, None]
        pn = (beta * q + bar) / (K * beta * q + bar.sum(1, keepdim=True))
        pi = torch.where(ok[:, None], pn, pi)
        mud = torch.where(live[..., None], new, mud)
        mux = torch.where(live[..., None], mux + m[..., 2:], mux)
        if case["accurate"]:
            W2, _, A0, _, A2 = _stats(x["off"], x["smp"], pi, mud, mux, cov)
            bar2 = A0 / Ws
            sig = (beta[..., None, None] * B + A2 / Ws[..., None, None]) / (beta * a + bar2)[..., None, None]
            s0n, s2n, can = A0, A2, live & (bar2 > 1e-12)
        else:
            s0n, s2n, can = hS0, TCT, live
        spd = torch.linalg.cholesky_ex(sig).info == 0
        cov = torch.where((can & spd)[..., None, None], sig, cov)
        s0 = torch.where(live if case["accurate"] else ok[:, None], s0n, s0)
        s2 = torch.where(live[..., None, None], s2n, torch.where(ok[:, None, None, None], hS2, s2))
        sw = torch.where(ok, hW, sw)
    return {"status": None, "table": None, "state": {"s0": s0.reshape(-1), "s2": _pack(s2).reshape(-1), "sw": sw, "step": None},
            "mix": {"pi": pi.reshape(-1), "mu_dir": mud.reshape(-1), "mu_pos": mux.reshape(-1),
                    "cov": _pack(cov).reshape(-1)}}


def _exact_grad(case, x):
    C, K = case["cells"], case["K"]
    pi, mud, mux, cov = _mixture64(x["mix"], C, K)
    off, smp = x["off"], x["smp"]
    beta, q, a = 1e-3, 1.0 / K, 5.0 / K
    B = torch.tensor([0.1, 0.1, 1.0, 1.0, 1.0], device=DEV, dtype=F64) * a * 1e-4
    leaf = [pi.log(), torch.zeros(C, K, 2, device=DEV, dtype=F64), mux.clone(), _pack(torch.linalg.cholesky(cov))]
    Fs, grads = [], [[] for _ in leaf]
    ends = off.tolist()
    lo = 0
    while lo < C:  # cells are independent: whole cells, about 2^20 pairs at a time
        hi = lo + 1
        while hi < C and (ends[hi + 1] - ends[lo]) * K <= 1 << 20:
            hi += 1
        p = [t[lo:hi].clone().requires_grad_(True) for t in leaf]
        L = torch.zeros(hi - lo, K, 5, 5, device=DEV, dtype=F64)
        for j, (d, e) in enumerate(_tri_index()):
            L[..., d, e] = p[3][..., j]
        Li = torch.linalg.solve_triangular(L, torch.eye(5, device=DEV, dtype=F64).expand_as(L), upper=False)
        lp = torch.log_softmax(p[0], -1)
        ld = L.diagonal(dim1=-2, dim2=-1).log().sum(-1)
        # exp about the directional mean at delta = 0, to second order in delta
        d2 = (p[1] * p[1]).sum(-1, keepdim=True)
        R = _frame(mud[lo:hi])
        v = torch.cat([p[1] * (1 - d2 / 6), 1 - d2 / 2], -1)
        mu = _unit((R * v.unsqueeze(-1)).sum(-2))
        fr = _frame(mu)
        cell = torch.repeat_interleave(torch.arange(hi - lo, device=DEV), off[lo + 1:hi + 1] - off[lo:hi])
        s = smp[:, ends[lo]:ends[hi]].to(F64)
        l, _ = _log_density(fr[cell], p[2][cell], Li[cell], (lp - ld - 2.5 * LOG2PI)[cell], s[0:3].T, s[3:6].T)
        W = torch.zeros(hi - lo, device=DEV, dtype=F64).index_add(0, cell, s[6])
        M = torch.zeros(hi - lo, device=DEV, dtype=F64).index_add(0, cell, (s[6] > 0).to(F64))
        ok = (M >= 16) & (W > 0)
        Wd = torch.where(ok, W, torch.ones_like(W))
        F = torch.zeros(hi - lo, device=DEV, dtype=F64).index_add(0, cell, s[6] / Wd[cell] * torch.logsumexp(l, -1))
        inv = (Li * Li * B[None, None, None, :]).sum((-1, -2))
        F = F + (beta * q * lp - beta * a * ld - 0.5 * beta * inv).sum(-1)
        F = torch.where(ok, F, torch.zeros_like(F))
        for acc, gr in zip(grads, torch.autograd.grad(F.sum(), p)):
            acc.append(gr)
        Fs.append(F.detach())
        lo = hi
    return {"F": torch.cat(Fs), "status": None, "grads": [torch.cat(v) for v in grads]}


def _exact_tree(case, x):
    n, K, cap = case["n"], case["K"], case["max_leaves"]
    smp = x["smp"]
    p = smp[3:6].to(F64)
    levels = 3 * case["depth"]
    side = 1 << case["depth"]
    L = side ** 3
    i = [(p[d] * side).floor().clamp(0, side - 1).long() for d in range(3)]
    leaf = torch.zeros(n, device=DEV, dtype=torch.int64)
    box = torch.arange(L, device=DEV)
    lo = torch.zeros(cap, 3, device=DEV, dtype=F64)
    hi = torch.zeros(cap, 3, device=DEV, dtype=F64)
    c = [torch.zeros(L, device=DEV, dtype=torch.int64) for _ in range(3)]
    for b in range(levels):  # the tree's order: x, y, z halvings in turn, left to right
        d, bit = b % 3, case["depth"] - 1 - b // 3
        leaf = leaf * 2 + ((i[d] >> bit) & 1)
        c[d] = c[d] * 2 + ((box >> (levels - 1 - b)) & 1)
    for d in range(3):
        lo[:L, d] = c[d].to(F64) / side
        hi[:L, d] = (c[d] + 1).to(F64) / side
    split = torch.zeros(2 * cap - 1, device=DEV, dtype=F64)
    node = torch.arange(L - 1, 2 * L - 1, device=DEV)  # node of each leaf
    for b in range(levels):
        first, m = (1 << b) - 1, 1 << b
        for k in range(min(m, 1 << 9)):
            path = [(k >> (b - 1 - j)) & 1 for j in range(b)]
            d, v = b % 3, 0.0
            for j, bit in enumerate(path):
                if j % 3 == d:
                    v += bit / (1 << (j // 3 + 1))
            split[first + k] = v + 0.5 / (1 << (b // 3))
    nodes, act = 2 * L - 1, torch.ones(L, device=DEV, dtype=torch.bool)
    while True:
        cnt = torch.bincount(leaf, minlength=L)
        s1 = torch.zeros(L, 3, device=DEV, dtype=F64).index_add_(0, leaf, p.T)
        s2 = torch.zeros(L, 3, device=DEV, dtype=F64).index_add_(0, leaf, p.T * p.T)
        mn = torch.full((L, 3), math.inf, device=DEV, dtype=F64)
        mx = -mn
        for d in range(3):
            mn[:, d] = mn[:, d].scatter_reduce(0, leaf, p[d], "amin")
            mx[:, d] = mx[:, d].scatter_reduce(0, leaf, p[d], "amax")
        mean = s1 / cnt.clamp_min(1)[:, None]
        ax = (s2 / cnt.clamp_min(1)[:, None] - mean * mean).max(1).indices
        r = torch.arange(L, device=DEV)
        sp = mean[r, ax]
        want = act & (cnt > case["split"]) & (mn[r, ax] < sp) & (sp <= mx[r, ax])
        who = want.nonzero().flatten()[: max(0, min(cap - L, cap - 1 - (nodes - 1) // 2))]
        if not who.numel():
            break
        new = torch.full((L,), -1, device=DEV, dtype=torch.int64)
        new[who] = L + torch.arange(who.numel(), device=DEV)
        at = torch.where(ax[leaf] == 0, p[0], torch.where(ax[leaf] == 1, p[1], p[2]))
        leaf = torch.where((new[leaf] >= 0) & (at >= sp[leaf]), new[leaf], leaf)
        nw = new[who]
        lo[nw], hi[nw] = lo[who], hi[who]
        hi[who, ax[who]] = sp[who]
        lo[nw, ax[who]] = sp[who]
        split[node[who]] = sp[who]
        kids = nodes + 2 * torch.arange(who.numel(), device=DEV)
        node = torch.cat([node, kids + 1])
        node[who] = kids
        nodes += 2 * who.numel()
        act = torch.zeros(L + who.numel(), device=DEV, dtype=torch.bool)
        act[who] = True
        act[nw] = True
        L += who.numel()
    order = torch.argsort(leaf, stable=True)
    got = (torch.bincount(leaf, minlength=L) >= 16)[:, None]
    m = _box_mixtures(lo[:L], hi[:L] - lo[:L], K)
    z = {k: torch.zeros(cap, v.numel() // L, device=DEV, dtype=F64) for k, v in m.items()}
    for k, v in m.items():
        z[k][:L] = torch.where(got, v.reshape(L, -1), z[k][:L])
    return {"sorted": smp[:, order], "offsets": None, "leaves": None, "status": None,
            "tree": {"split": split, "lo": lo, "hi": hi}, "mix": {k: v.reshape(-1) for k, v in z.items()},
            "state": {"s0": torch.zeros(cap * K, device=DEV, dtype=F64), "s2": torch.zeros(cap * K * 15, device=DEV, dtype=F64),
                      "sw": torch.zeros(cap, device=DEV, dtype=F64)}}


def _conditional(mix, C, K):
    """What conditioning on the last three coordinates needs of every component."""
    pi, mud, mux, cov = _mixture64(mix, C, K)
    xx, nx = cov[..., 2:, 2:], cov[..., :2, 2:]
    A = torch.linalg.solve(xx, nx.mT).mT
    L = torch.linalg.cholesky(xx)
    cc = cov[..., :2, :2] - A @ nx.mT
    return {"R": _frame(mud), "mux": mux, "A": A,
            "Lxi": torch.linalg.solve_triangular(L, torch.eye(3, device=DEV, dtype=F64).expand_as(L), upper=False),
            "lw": pi.log() - L.diagonal(dim1=-2, dim2=-1).log().sum(-1), "L": torch.linalg.cholesky(cc)}


def _at(t, cell, x):
    """Conditioned weights (log), means, and the components' frames and factors at x [n, 3]."""
    d = x[:, None] - t["mux"][cell]
    z = (t["Lxi"][cell] * d.unsqueeze(-2)).sum(-1)
    lw = torch.log_softmax(t["lw"][cell] - 0.5 * (z * z).sum(-1), -1)
    return lw, (t["A"][cell] * d.unsqueeze(-2)).sum(-1), t["R"][cell], t["L"][cell]


def _gauss2(L, d):
    """log N2 density at offsets d [..., 2] with factor L [..., 2, 2]."""
    z0 = d[..., 0] / L[..., 0, 0]
    z1 = (d[..., 1] - L[..., 1, 0] * z0) / L[..., 1, 1]
    return -0.5 * (z0 * z0 + z1 * z1) - (L[..., 0, 0] * L[..., 1, 1]).log() - LOG2PI


CUT = math.pi * (1 - 1e-6)


def _pdf(lw, m, R, L, w):
    """Solid-angle density at directions w [n, t, 3]."""
    nu, f, _ = _log(R[:, None], w[:, :, None])
    p = torch.exp(lw[:, None] + _gauss2(L[:, None], nu - m[:, None])) * f
    return torch.where(nu.norm(dim=-1) < CUT, p, torch.zeros_like(p)).sum(-1)


def _philox(n0, n1, seed):
    """Philox4x32-10 uniforms of draws n0..n1-1 (counter = draw index): [3, n]."""
    mask = 0xFFFFFFFF

    def mul(a, b):
        t = a * (b & 0xFFFF)
        return ((a * (b >> 16) + (t >> 16)) >> 16) & mask, (t + ((a * (b >> 16)) << 16)) & mask

    i = torch.arange(n0, n1, device=DEV, dtype=torch.int64)
    c = [i & mask, i >> 32, torch.zeros_like(i), torch.zeros_like(i)]
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return torch.stack([(v >> 8).to(F64) * 2.0 ** -24 for v in c[:3]])


def _uniforms(x, total, a, b):
    u = x["u"][:, a:b].to(F64) if x["u"] is not None else _philox(a, b, x["seed"])
    return u


def _draw(w, m, R, L, u):
    """ns draws per row from components of probability w [n, K] (u [3, n, ns]): the
    component, the direction and whether it lies inside the cut locus."""
    cdf = w.cumsum(-1)
    k = torch.searchsorted(cdf, u[0].contiguous(), right=True)
    last = (w > 0).to(torch.int64).mul(torch.arange(1, w.shape[1] + 1, device=DEV)).max(-1).values - 1
    k = torch.minimum(k, last[:, None]).clamp_min(0)
    row = torch.arange(w.shape[0], device=DEV)[:, None]
    rad, ang = torch.sqrt(-2 * torch.log1p(-u[1])), 2 * math.pi * u[2]
    z = torch.stack([rad * torch.cos(ang), rad * torch.sin(ang)], -1)
    nu = m[row, k] + (L[row, k] * z.unsqueeze(-2)).sum(-1)
    return k, _exp(R[row, k], nu), nu.norm(dim=-1) < math.pi


def _chunks(n, K, ns):
    step = max(1, (1 << 22) // (K * max(1, ns)))
    return [(a, min(n, a + step)) for a in range(0, n, step)]


def _exact_guide(case, x):
    C, K, nq, ns = case["cells"], case["K"], case["nq"], case["ns"]
    t = _conditional(x["mix"], C, K)
    nd = nq * ns
    out = {"dirs": torch.empty(3, nd, device=DEV, dtype=F64), "pdf": torch.empty(nd, device=DEV, dtype=F64)}
    mis = case["op"] == "mis"
    if mis:
        ne = case["nd"]
        out |= {"weights": torch.empty(nq, K, device=DEV, dtype=F64), "means": torch.empty(nq, K, 2, device=DEV, dtype=F64),
                "other": torch.empty(nq * ne, device=DEV, dtype=F64)}
    for a, b in _chunks(nq, K, max(ns, case.get("nd", 1))):
        lw, m, R, L = _at(t, x["qcell"][a:b].long(), x["qpos"][:, a:b].T.to(F64))
        u = _uniforms(x, nd, a * ns, b * ns).reshape(3, b - a, ns)
        _, w, ok = _draw(lw.exp(), m, R, L, u)
        p = _pdf(lw, m, R, L, w)
        out["dirs"][:, a * ns:b * ns] = (w * ok[..., None]).reshape(-1, 3).T
        out["pdf"][a * ns:b * ns] = (p * ok).reshape(-1)
        if mis:
            out["weights"][a:b], out["means"][a:b] = lw.exp(), m
            e = x["dirs"][:, a * ne:b * ne].T.to(F64).reshape(b - a, ne, 3)
            out["other"][a * ne:b * ne] = _pdf(lw, m, R, L, e).reshape(-1)
    return out | {"valid": None} | ({"comp": None} if mis else {})


def _exact_product(case, x):
    C, K, Kb, nq, ns, ne = (case[k] for k in ("cells", "K", "Kb", "nq", "ns", "nd"))
    t, tb = _conditional(x["mix"], C, K), _conditional(x["bmix"], case["models"], Kb)
    nd = nq * ns
    out = {"dirs": torch.empty(3, nd, device=DEV, dtype=F64), "pdf": torch.empty(nd, device=DEV, dtype=F64),
           "other": torch.empty(nq * ne, device=DEV, dtype=F64), "valid": None}
    for a, b in _chunks(nq, 2 * K, 2 * max(ns, ne)):
        n = b - a
        row = torch.arange(n, device=DEV)[:, None]
        lw, m, R, L = _at(t, x["qcell"][a:b].long(), x["qpos"][:, a:b].T.to(F64))
        bw, bm, bR, bL = _at(tb, x["bcell"][a:b].long(), x["bpar"][:, a:b].T.to(F64))
        top = bw.topk(min(2, Kb), dim=-1).indices  # the two heaviest
        F = x["frames"][:, a:b].T.to(F64).reshape(n, 1, 3, 3)
        Rw = bR[row, top] @ F.mT  # rows F t1, F t2, F mu
        bn, bl = bm[row, top], bL[row, top]
        centre = _exp(Rw, bn)
        D = Rw.mT @ _exp_jacobian(bn)  # 3 x 2
        # every pair (k, j) in the tangent space of mu_k
        nu, f, v = _log(R[:, :, None], centre[:, None])
        px, py, pz = v.unbind(-1)
        s2 = px * px + py * py
        g = torch.where(s2 > 1e-10, (pz - f) / s2.clamp_min(1e-10), torch.full_like(s2, -2.0 / 3))
        Jl = torch.stack([torch.stack([f + px * px * g, px * py * g, -px], -1),
                          torch.stack([px * py * g, f + py * py * g, -py], -1)], -2)
        J = Jl @ (R[:, :, None] @ D[:, None])
        Bc = J @ (bl @ bl.mT)[:, None] @ J.mT
        Ac = (L @ L.mT)[:, :, None]
        S = Ac + Bc
        d = m[:, :, None] - nu
        Si = torch.linalg.inv(S)
        q = (d.unsqueeze(-2) @ Si @ d.unsqueeze(-1))[..., 0, 0]
        lam = lw[:, :, None] + bw[row, top][:, None] - 0.5 * q - LOG2PI - 0.5 * torch.linalg.det(S).log()
        Cc = Ac @ Si @ Bc
        Lc = torch.linalg.cholesky_ex(0.5 * (Cc + Cc.mT)).L
        cm = m[:, :, None] - (Ac @ Si @ d.unsqueeze(-1))[..., 0]
        P = 2 if Kb > 1 else 1
        lp = torch.log_softmax(lam.reshape(n, K * P), -1)
        mm, LL = cm.reshape(n, K * P, 2), Lc.reshape(n, K * P, 2, 2)
        RR = R[:, :, None].expand(n, K, P, 3, 3).reshape(n, K * P, 3, 3)
        u = _uniforms(x, nd, a * ns, b * ns).reshape(3, n, ns)
        _, w, ok = _draw(lp.exp(), mm, RR, LL, u)
        out["dirs"][:, a * ns:b * ns] = (w * ok[..., None]).reshape(-1, 3).T
        out["pdf"][a * ns:b * ns] = (_pdf(lp, mm, RR, LL, w) * ok).reshape(-1)
        e = x["dirs"][:, a * ne:b * ne].T.to(F64).reshape(n, ne, 3)
        out["other"][a * ne:b * ne] = _pdf(lp, mm, RR, LL, e).reshape(-1)
    return out


def exact(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    if op == "fit":
        return _exact_fit(case, x)
    if op == "grad":
        return _exact_grad(case, x)
    if op == "tree":
        return _exact_tree(case, x)
    return _exact_product(case, x) if op == "product" else _exact_guide(case, x)
