"""Workloads of the Viterbi decoders, from the smallest call to the largest batch.

Each case is a call (or a training step) that a program makes through the
package's entry points, at sizes of this repository's benchmark, tests and
sweeps, odd sizes among them.  Inputs follow the distributions of the seeded
workloads in workloads/hmm.py (log-Dirichlet or Erdos-Renyi transitions,
discrete, Gaussian or network emissions, a road-like sparse graph), drawn here
on the device so that the large ones are quick to make.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_19301_amd as fv

F32 = torch.float32
F64 = torch.float64


def listed():
    return [
        # one short observation sequence on a small model: an interactive
        # request, where the launches and the host path count
        {"name": "short_k32_vanilla", "kind": "discrete", "method": "vanilla", "K": 32, "V": 50, "n": 1,
         "t_lo": 32, "t_hi": 32, "P": 1, "B": 0},
        # the discrete HMM of the benchmark: symbols to scores to path
        {"name": "discrete_k64_flash", "kind": "discrete", "method": "flash", "K": 64, "V": 128, "n": 1,
         "t_lo": 1000, "t_hi": 1000, "P": 16, "B": 0},
        # many sequences on one small model: a server's batch of requests
        {"name": "discrete_batch_k64_vanilla", "kind": "discrete", "method": "vanilla", "K": 64, "V": 128, "n": 256,
         "t_lo": 200, "t_hi": 1000, "P": 1, "B": 0},
        # one sequence on an Erdos-Renyi graph, the default point of the sweeps
        {"name": "er_k512_flash", "kind": "er", "method": "flash", "K": 512, "V": 50, "n": 1,
         "t_lo": 512, "t_hi": 512, "P": 16, "B": 0},
        # structured-prediction training step: decode, then the score's gradients
        {"name": "crf_k256_step", "kind": "crf", "method": "flash", "K": 256, "n": 512,
         "t_lo": 32, "t_hi": 512, "P": 16, "B": 0},
        # the headline workload: FLASH over 256 sequences of very uneven length
        {"name": "batch_k1024_flash", "kind": "dense", "method": "flash", "K": 1024, "n": 256,
         "t_lo": 500, "t_hi": 8000, "P": 64, "B": 0, "alpha": 0.1, "sigma": 2.0},
        # a smaller batch, vanilla, at a state count that is no multiple of a tile
        {"name": "batch_k1000_vanilla", "kind": "dense", "method": "vanilla", "K": 1000, "n": 64,
         "t_lo": 100, "t_hi": 2000, "P": 1, "B": 0, "alpha": 0.1, "sigma": 2.0},
        # beam decoding of a batch
        {"name": "batch_k1024_beam", "kind": "dense", "method": "beam", "K": 1024, "n": 64,
         "t_lo": 200, "t_hi": 2000, "P": 16, "B": 64, "alpha": 0.1, "sigma": 2.0},
        # one sequence on a very large dense model (log A of 1 GiB)
        {"name": "large_k16384_vanilla", "kind": "dense", "method": "vanilla", "K": 16384, "n": 1,
         "t_lo": 512, "t_hi": 512, "P": 1, "B": 0, "alpha": 0.05, "sigma": 3.0},
        # one sequence on a large dense model of odd size, in little memory
        {"name": "large_k5001_flash", "kind": "dense", "method": "flash", "K": 5001, "n": 1,
         "t_lo": 777, "t_hi": 777, "P": 16, "B": 0, "alpha": 0.05, "sigma": 3.0},
        # map matching: trajectories on a sparse road-like graph, emission
        # scores generated from the GPS points, exact and with a beam
        {"name": "map_k99856_flash", "kind": "map", "method": "flash", "K": 99856, "n": 32,
         "t_lo": 100, "t_hi": 600, "P": 16, "B": 0},
        {"name": "map_k99856_beam", "kind": "map", "method": "beam", "K": 99856, "n": 64,
         "t_lo": 200, "t_hi": 2000, "P": 16, "B": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["discrete", "discrete_batch", "er", "crf", "dense_batch", "dense_batch", "beam", "large", "map"])
    exact = rng.choice(["vanilla", "flash"])
    P = rng.choice([4, 16, 64])
    if kind == "discrete":
        T = _log_int(rng, 16, 2000)
        return {"kind": "discrete", "method": exact, "K": _log_int(rng, 8, 256), "V": _log_int(rng, 16, 128), "n": 1,
                "t_lo": T, "t_hi": T, "P": P, "B": 0}
    if kind == "discrete_batch":
        T = _log_int(rng, 64, 1000)
        return {"kind": "discrete", "method": exact, "K": _log_int(rng, 16, 128), "V": _log_int(rng, 16, 128),
                "n": _log_int(rng, 2, 512), "t_lo": max(1, T // 5), "t_hi": T, "P": P, "B": 0}
    if kind == "er":
        T = _log_int(rng, 32, 1024)
        return {"kind": "er", "method": exact, "K": _log_int(rng, 32, 2048), "V": 50, "n": 1, "t_lo": T, "t_hi": T,
                "P": P, "B": 0}
    if kind == "crf":
        T = _log_int(rng, 32, 512)
        return {"kind": "crf", "method": exact, "K": _log_int(rng, 16, 256), "n": _log_int(rng, 8, 512),
                "t_lo": max(1, T // 16), "t_hi": T, "P": P, "B": 0}
    if kind == "dense_batch":
        T = _log_int(rng, 200, 2000)
        return {"kind": "dense", "method": exact, "K": _log_int(rng, 300, 2048), "n": _log_int(rng, 2, 128),
                "t_lo": max(1, T // 16), "t_hi": T, "P": P, "B": 0, "alpha": 0.1, "sigma": 2.0}
    if kind == "beam":
        T = _log_int(rng, 100, 1000)
        return {"kind": "dense", "method": "beam", "K": _log_int(rng, 300, 2048), "n": _log_int(rng, 1, 64),
                "t_lo": max(1, T // 10), "t_hi": T, "P": 16, "B": _log_int(rng, 16, 256), "alpha": 0.1, "sigma": 2.0}
    if kind == "large":
        T = _log_int(rng, 64, 512)
        return {"kind": "dense", "method": exact, "K": _log_int(rng, 4100, 16384), "n": 1, "t_lo": T, "t_hi": T,
                "P": P, "B": 0, "alpha": 0.05, "sigma": 3.0}
    side = _log_int(rng, 64, 316)
    T = _log_int(rng, 60, 600)
    method = rng.choice(["vanilla", "flash", "beam"])
    return {"kind": "map", "method": method, "K": side * side, "n": _log_int(rng, 1, 32), "t_lo": max(1, T // 6),
            "t_hi": T, "P": 16, "B": 128 if method == "beam" else 0}


# ------------------------------------------------------------------ inputs
def _lengths(case):
    """The case's sequence lengths (they belong to its sizes: no seed)."""
    n, lo, hi = case["n"], case["t_lo"], case["t_hi"]
    return np.random.default_rng([n, lo, hi]).integers(lo, hi + 1, size=n).astype(np.int32)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _log_dirichlet(g, rows, cols, alpha):
    """float32 [rows, cols] on the device: every row is the log of a Dirichlet(alpha) draw."""
    out = torch.empty((rows, cols), dtype=F32, device="cuda")
    step = max(1, (1 << 24) // cols)
    for r in range(0, rows, step):
        m = min(step, rows - r)
        a = torch.full((m, cols), alpha + 1.0, dtype=F32, device="cuda")
        u = torch.rand((m, cols), generator=g, dtype=F32, device="cuda").clamp_min_(1e-38).to(F64)
        x = torch._standard_gamma(a, generator=g).to(F64).log_() + u.log_() / alpha
        out[r:r + m] = (x - torch.logsumexp(x, 1, keepdim=True)).to(F32)
    return out


def _observations(rng, log_a, log_e, n, T):
    """int32 [n, T] symbols of n walks through the model."""
    pa = np.cumsum(np.exp(log_a.double().cpu().numpy()), axis=1)
    pe = np.cumsum(np.exp(log_e.double().cpu().numpy()), axis=1)
    K, V = log_e.shape
    obs = np.empty((n, T), np.int32)
    q = rng.integers(0, K, size=n)
    for t in range(T):
        obs[:, t] = np.minimum((pe[q] < rng.random((n, 1))).sum(1), V - 1)
        q = np.minimum((pa[q] < rng.random((n, 1))).sum(1), K - 1)
    return torch.from_numpy(obs).cuda()


def _grid_graph(g, side):
    """A road-like sparse graph: side x side jittered points of the unit
    square, each with the nine points around it (itself among them)."""
    K = side * side
    c = torch.arange(side, device="cuda")
    y, x = torch.meshgrid(c, c, indexing="ij")
    cell = torch.stack([x.reshape(-1), y.reshape(-1)], 1).to(F64)
    xy = ((cell + torch.rand((K, 2), generator=g, dtype=F64, device="cuda")) / side).contiguous()
    x0 = (x.reshape(-1) - 1).clamp(0, side - 3)
    y0 = (y.reshape(-1) - 1).clamp(0, side - 3)
    off = torch.arange(3, device="cuda")
    col = ((y0[:, None, None] + off[None, :, None]) * side + x0[:, None, None] + off[None, None, :]).reshape(K, 9)
    dist = (xy[col] - xy[:, None, :]).square().sum(2).sqrt()
    val = torch.log_softmax(-dist * (side / 3.16), 1).to(F32).contiguous()
    row_ptr = (torch.arange(K + 1, device="cuda") * 9).to(torch.int32)
    return xy, row_ptr, col.to(torch.int32).contiguous(), val


def _inputs(case, seed):
    """Everything a case is made of, on the device."""
    g = _generator(seed)
    rng = np.random.default_rng(seed)
    K, n, lens = case["K"], case["n"], _lengths(case)
    s = {"lengths": lens, "log_pi": torch.full((K,), -math.log(K), dtype=F32, device="cuda")}
    kind = case["kind"]
    if kind in ("discrete", "er"):
        if kind == "er":
            mask = torch.rand((K, K), generator=g, device="cuda") < 0.253
            eye = torch.eye(K, dtype=torch.bool, device="cuda")
            mask |= eye & ~mask.any(1, keepdim=True)
            w = torch.where(mask, 1.0 - torch.rand((K, K), generator=g, dtype=F64, device="cuda"), 0.0)
            s["log_a"] = (w / w.sum(1, keepdim=True)).log().to(F32)
            s["log_e"] = _log_dirichlet(g, K, case["V"], 1.0)
        else:
            s["log_a"] = _log_dirichlet(g, K, K, 1.0)
            s["log_e"] = _log_dirichlet(g, K, case["V"], 0.5)
        s["obs"] = _observations(rng, s["log_a"], s["log_e"], n, int(lens.max()))
    elif kind == "crf":
        tmax = int(lens.max())
        bound = 1.0 / math.sqrt(512)
        w = (torch.rand((512, K), generator=g, device="cuda") * 2 - 1) * bound
        b = (torch.rand((K,), generator=g, device="cuda") * 2 - 1) * bound
        em = torch.zeros((n, tmax, K), dtype=F32, device="cuda")
        for k in range(n):
            em[k, :lens[k]] = torch.randn((int(lens[k]), 512), generator=g, device="cuda") @ w + b
        s["emissions"] = em
        s["log_a"] = torch.randn((K, K), generator=g, device="cuda") * 0.1
        s["grad"] = torch.randn((n,), generator=g, device="cuda")
        s["log_pi"] = None
    elif kind == "dense":
        s["log_a"] = _log_dirichlet(g, K, K, case["alpha"])
        s["log_b"] = [torch.randn((int(T), K), generator=g, device="cuda") * case["sigma"] for T in lens]
    else:
        side = math.isqrt(K)
        xy, row_ptr, col, val = _grid_graph(g, side)
        sigma = 0.005 * 316 / side
        T = int(lens.max())
        walk = np.empty((T, n), np.int64)
        nb = col.cpu().numpy()
        q = rng.integers(0, K, size=n)
        for t in range(T):
            walk[t] = q
            q = nb[q, rng.integers(0, 9, size=n)]
        pts = xy[torch.from_numpy(walk).cuda()]
        pts = pts + torch.randn(pts.shape, generator=g, dtype=F64, device="cuda") * sigma
        s.update(xy=xy, row_ptr=row_ptr, col=col.reshape(-1), val=val.reshape(-1), sigma=sigma,
                 obs=[pts[:int(lens[b]), b].contiguous() for b in range(n)])
    return s


# ------------------------------------------------------------------ what a program holds, and one pass
def prepare(case, seed):
    s = _inputs(case, seed)
    kind, n = case["kind"], case["n"]
    st = {"case": case, "log_pi": s["log_pi"], "ws": None}
    if kind in ("discrete", "er"):
        st["log_a"], st["log_e"], st["lengths"] = s["log_a"], s["log_e"], s["lengths"]
        st["obs"] = [s["obs"][b, :int(T)].contiguous() for b, T in enumerate(s["lengths"])]
        st["log_b"] = [torch.empty((int(T), case["K"]), dtype=F32, device="cuda") for T in s["lengths"]]
        if n > 1:
            # a batch's scores are on the device before the decode
            for b in range(n):
                _gather(st, b)
            st["batch"] = fv.Batch(st["log_b"])
    elif kind == "crf":
        st["emissions"] = s["emissions"].requires_grad_(True)
        st["transitions"] = s["log_a"].requires_grad_(True)
        st["lengths"], st["grad"] = s["lengths"], s["grad"]
    elif kind == "dense":
        st["log_a"] = s["log_a"]
        if n > 1:
            st["batch"] = fv.Batch(s["log_b"])
        else:
            st["log_b"] = s["log_b"]
    else:
        st["log_a"] = fv.CsrModel(s["row_ptr"], s["col"], s["val"])
        st["emission"] = fv.GaussEmission.from_sigma(s["xy"], s["sigma"])
        st["batch"] = fv.Batch.observations(s["obs"])
    return st


def _gather(st, b):
    """Scores of sequence b's symbols (fv_gather_emissions of the C interface)."""
    K, V = st["log_e"].shape
    T = int(st["lengths"][b])
    rc = fv.lib().fv_gather_emissions(K, V, st["log_e"].data_ptr(), st["obs"][b].data_ptr(), T,
                                      st["log_b"][b].data_ptr(), K, torch.cuda.current_stream().cuda_stream)
    if rc != fv.FV_OK:
        raise RuntimeError(f"fv_gather_emissions: status {rc}")


def run(st):
    c = st["case"]
    if c["kind"] == "crf":
        st["emissions"].grad = None
        st["transitions"].grad = None
        scores, paths = fv.ViterbiScore.apply(st["emissions"], st["lengths"], st["transitions"], None, c["method"],
                                              c["P"])
        scores.backward(st["grad"])
        return {"scores": scores.detach(), "paths": paths, "grad_emissions": st["emissions"].grad,
                "grad_transitions": st["transitions"].grad}
    if c["n"] == 1 and c["kind"] != "map":
        if c["kind"] in ("discrete", "er"):
            _gather(st, 0)
        path, score, status = fv.decode(st["log_a"], st["log_b"][0], st["log_pi"], c["method"], P=c["P"], B=c["B"])
        return {"scores": score, "paths": path, "status": status}
    b = st["batch"]
    st["ws"] = fv.decode_batch(st["log_a"], b, st["log_pi"], method=c["method"], P=c["P"], B=c["B"], ws=st["ws"],
                               emission=st.get("emission"))
    return {"scores": b.scores, "paths": b.paths, "status": b.status}


# ------------------------------------------------------------------ the work
def work(case):
    """Inputs read once, outputs written once; the recurrence's operations:
    an addition and a comparison per candidate."""
    K, lens = case["K"], _lengths(case).astype(np.int64)
    total, steps, n, tmax = int(lens.sum()), int((lens - 1).sum()), case["n"], int(lens.max())
    out = 4 * total + 8 * n
    beam = case["method"] == "beam" and case["B"] < K
    if case["kind"] == "map":
        edges = 9 * K
        per_step = 9 * case["B"] if beam else edges
        return {"bytes": out + 16 * total + 8 * edges + 20 * K, "flops": 2 * steps * per_step}
    per_step = case["B"] * K if beam else K * K
    model = 4 * K * K + 4 * K
    if case["kind"] in ("discrete", "er") and n == 1:
        scores = 4 * K * case["V"] + 4 * total
    else:
        scores = 4 * K * total
    grads = (4 * n * tmax * K + 4 * K * K) if case["kind"] == "crf" else 0
    return {"bytes": out + model + scores + grads, "flops": 2 * steps * per_step}


# ------------------------------------------------------------------ 64 bits
def _viterbi64(log_a, log_pi, log_b, lens, paths=False):
    """float64 scores [n] (and decoded paths) of log_b [n, Tmax, K], every sequence at once."""
    n, tmax, K = log_b.shape
    a = log_a.to(F64).t().contiguous()          # a[j, i]
    d = log_b[:, 0].to(F64) + (0.0 if log_pi is None else log_pi.to(F64))
    last = d.clone()
    lens_t = torch.from_numpy(np.asarray(lens, np.int64)).to(log_b.device)
    psi = torch.zeros((tmax, n, K), dtype=torch.int16, device=log_b.device) if paths else None
    rows = max(1, (1 << 28) // (K * K))
    for t in range(1, tmax):
        live = torch.nonzero(lens_t > t).reshape(-1)
        new = torch.empty((live.numel(), K), dtype=F64, device=log_b.device)
        for r in range(0, live.numel(), rows):
            idx = live[r:r + rows]
            m, arg = (d[idx][:, None, :] + a[None]).max(2)
            new[r:r + rows] = m
            if paths:
                psi[t, idx] = arg.to(torch.int16)
        d[live] = new + log_b[live, t].to(F64)
        last[live] = d[live]
    score, q = last.max(1)
    if not paths:
        return score, None
    out = torch.full((n, tmax), -1, dtype=torch.int64, device=log_b.device)
    ar = torch.arange(n, device=log_b.device)
    for t in range(tmax - 1, -1, -1):
        on = lens_t > t
        out[on, t] = q[on]
        if t:
            q = torch.where(on, psi[t][ar, q].to(torch.int64) & 0x7fff, q)
    return score, out


def exact(case, seed):
    """Scores (and gradients) in 64 bits; paths are whole numbers and a beam's
    score depends on its pruning: None in their place."""
    K, lens = case["K"], _lengths(case)
    none = {"scores": None, "paths": None, "status": None}
    if case["kind"] == "crf":
        none = {"scores": None, "paths": None, "grad_emissions": None, "grad_transitions": None}
    tmax, n = int(lens.max()), case["n"]
    candidates = float((lens.astype(np.int64) - 1).sum()) * K * K
    if case["kind"] == "map" or case["method"] == "beam" or candidates > 3e11:
        return None
    s = _inputs(case, seed)
    if case["kind"] in ("discrete", "er"):
        log_b = s["log_e"].t()[s["obs"].long()]
    elif case["kind"] == "crf":
        log_b = s["emissions"]
    else:
        log_b = torch.zeros((n, tmax, K), dtype=F32, device="cuda")
        for b, x in enumerate(s["log_b"]):
            log_b[b, :x.shape[0]] = x
    score, path = _viterbi64(s["log_a"], s["log_pi"], log_b, lens, paths=case["kind"] == "crf")
    out = dict(none, scores=score)
    if case["kind"] == "crf":
        g = s["grad"].to(F64)
        ge = torch.zeros((n, tmax, K), dtype=F64, device="cuda")
        ga = torch.zeros((K * K,), dtype=F64, device="cuda")
        on = path >= 0
        b, t = torch.nonzero(on, as_tuple=True)
        ge[b, t, path[b, t]] = g[b]
        b, t = torch.nonzero(on[:, 1:], as_tuple=True)
        ga.index_add_(0, path[b, t] * K + path[b, t + 1], g[b])
        out.update(grad_emissions=ge, grad_transitions=ga.reshape(K, K))
    return out
