"""The work that a user of this decoder has it do, as cases that can be timed.

Codes are the triangular 6.6.6 colour codes of synth/ at the sizes that the
benchmark and the tests run: code capacity (d = 3, 5, 7), phenomenological
(11 noisy rounds, d = 11) and circuit level (d rounds, d = 3 to 13, p = 1e-3).
A case names one entry point:

  decode    Graph.decode: the whole online stage (BP ensemble, selection, LSD)
  packed    Graph.decode_packed: the same from bit-packed syndromes
  ensemble  Graph.bp_ensemble: the members' posteriors, convergence iterations
            and decisions, without selection and LSD
  lsd       Graph.lsd: localised statistics decoding on given soft information
  ragged    Runtime.decode: requests on several codes as one call
  grad      Graph.bp_grad: loss and gradient through K unrolled iterations

Schedules are serial (the production setting), parallel (one member: the
BP+LSD-0 baseline) and layered; messages are 32 bits, or 64 for verification.
The member schedules belong to the graph and are fixed; the syndromes are
drawn from the seed.  Outputs are whole, except that the per-shot records
leave out the two fields that count work done before the correction limit
stopped the remaining members: those depend on timing from run to run.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2508_15743_amd as P
from synth.dem import circuit_dem, code_capacity_dem, phenomenological_dem
from synth.sample import permutations

# decoder settings of each code: members, correction limit, iterations
SETTINGS = {"capacity": (16, 5, 32), "phenom": (32, 5, 50), "circuit": (32, 5, 20), "circuit13": (64, 7, 25)}
# share of the iterations that a member runs before it converges or the
# correction limit stops it, measured per family (parallel: the one member)
RUN_SHARE = {"capacity": 0.2, "phenom": 0.45, "circuit": 0.63, "circuit13": 0.87}


@functools.lru_cache(maxsize=None)
def model(code, d):
    if code == "capacity":
        return code_capacity_dem(d, 0.05)
    if code == "phenom":
        return phenomenological_dem(d, d, 0.01, 0.01)
    return circuit_dem(d, d, 1e-3)


def settings(case, d=None):
    code, d = case["code"], d or case["d"]
    L, M, T = SETTINGS["circuit13" if code == "circuit" and d >= 13 else code]
    if case.get("schedule") == "parallel":
        L = M = 1
    return case.get("L", L), case.get("M", min(M, case.get("L", L))), T


def listed():
    return [
        # one shot of a small code: the cost of a call, nothing else
        {"name": "capacity d5, 1 shot", "path": "decode", "code": "capacity", "d": 5, "shots": 1},
        # one window of a memory experiment, decoded as it arrives
        {"name": "circuit d9, 1 shot", "path": "decode", "code": "circuit", "d": 9, "shots": 1},
        # the benchmark's latency batch
        {"name": "circuit d9, 64 shots", "path": "decode", "code": "circuit", "d": 9, "shots": 64},
        # the benchmark's throughput workload, in a batch that still fills the GPU many times over
        {"name": "circuit d9, 4096 shots", "path": "decode", "code": "circuit", "d": 9, "shots": 4096},
        # the largest code of the ragged and serving mixes, in a batch of odd size
        {"name": "circuit d13, 37 shots", "path": "decode", "code": "circuit", "d": 13, "shots": 37},
        # logical error rates of the phenomenological workload as configured, LSD order 10
        {"name": "phenom d11, 10007 shots", "path": "decode", "code": "phenom", "d": 11, "shots": 10007, "order": 10},
        # the code-capacity workload, from packed syndromes
        {"name": "capacity d5, 10000 packed", "path": "packed", "code": "capacity", "d": 5, "shots": 10000},
        # posteriors of every member, for studies of the ensemble
        {"name": "circuit d5 ensemble", "path": "ensemble", "code": "circuit", "d": 5, "shots": 20},
        # the baseline without an ensemble
        {"name": "circuit d9 parallel", "path": "decode", "code": "circuit", "d": 9, "shots": 8192, "schedule": "parallel"},
        # check-serial members
        {"name": "circuit d9 layered", "path": "decode", "code": "circuit", "d": 9, "shots": 200, "schedule": "layered"},
        # one step of fitting the channel LLRs and scaling factors
        {"name": "circuit d5 gradient", "path": "grad", "code": "circuit", "d": 5, "shots": 1024, "K": 16},
        # a round of requests on several codes
        {"name": "circuit d5 to d11 ragged", "path": "ragged", "code": "circuit", "d": 11, "shots": 128},
    ]


# Cost of a case in edge-updates, the unit that bounds the draws: about the
# largest listed decode (the slower paths are weighted by what they cost).
MOST = 1.0e11


def edge_updates(case):
    """Edge-updates of one pass, with the measured share of the iterations."""
    code = case["code"]
    if case["path"] == "lsd":
        return 0.0
    ds = [5, 7, 9, 11][: (case["d"] - 3) // 2] if case["path"] == "ragged" else [case["d"]]
    total = 0.0
    for d in ds:
        L, _, T = settings(case, d)
        share = 0.9 if case.get("schedule") == "parallel" else RUN_SHARE["circuit13" if code == "circuit" and d >= 13 else code]
        its = case["K"] if case["path"] == "grad" else max(1.0, share * T)
        total += float(case["shots"]) * L * its * model(code, d).nnz
    return total


def draw(rng):
    path = rng.choice(["decode", "decode", "decode", "decode", "packed", "ensemble", "lsd", "ragged", "grad"])
    code = rng.choice(["circuit", "circuit", "circuit", "phenom", "capacity"])
    if path in ("ragged", "grad", "ensemble", "lsd"):
        code = "circuit"
    d = rng.choice({"circuit": [3, 5, 7, 9, 11, 13], "phenom": [5, 7, 9, 11], "capacity": [3, 5, 7]}[code])
    case = {"path": path, "code": code, "d": d}
    weight = 1.0
    if path == "decode":
        kind = rng.random()
        if kind < 0.12:
            case["schedule"], weight = "parallel", 2.0
        elif kind < 0.24:
            case["schedule"], weight = "layered", 8.0
        elif kind < 0.36:
            case["bits"], weight = 64, 4.0
        elif kind < 0.5:
            case["order"] = rng.choice([1, 2, 10])
    elif path == "ragged":
        case["d"] = rng.choice([7, 9, 11])
    elif path == "grad":
        case["d"] = rng.choice([3, 5, 7])
        case["K"] = rng.choice([4, 8, 16])
        weight = 12.0
    elif path == "ensemble":
        case["d"] = rng.choice([3, 5, 7, 9])
    one = edge_updates(dict(case, shots=1))
    top = {"lsd": 2000.0, "ensemble": min(400.0, MOST / max(one, 1.0))}.get(path, MOST / max(one * weight, 1.0))
    case["shots"] = max(1, int(math.exp(rng.uniform(0.0, math.log(max(2.0, min(top, 20000.0)))))))
    return case


# ---------------------------------------------------------------- inputs


@functools.lru_cache(maxsize=8)
def dense(code, d):
    """H as a float matrix [n, m] and the priors, on the GPU, for the sampler."""
    dem = model(code, d)
    h = torch.zeros((dem.n, dem.m))
    rows = np.repeat(np.arange(dem.m), np.diff(dem.h_indptr.astype(np.int64)))
    h[torch.from_numpy(dem.h_indices.astype(np.int64)), torch.from_numpy(rows)] = 1.0
    return h.cuda(), torch.from_numpy(dem.priors.astype(np.float32)).cuda()


def syndromes(code, d, shots, seed):
    """Every mechanism fires with its prior; s = H e mod 2."""
    h, p = dense(code, d)
    gen = torch.Generator(device="cuda").manual_seed(seed * 1009 + d)
    out = torch.empty((shots, h.shape[1]), dtype=torch.uint8, device="cuda")
    for a in range(0, shots, 1024):
        b = min(shots, a + 1024)
        e = (torch.rand((b - a, h.shape[0]), generator=gen, device="cuda") < p).float()
        out[a:b] = torch.remainder(torch.matmul(e, h), 2.0).round().to(torch.uint8)
    return out


def graph(case, d=None):
    d = d or case["d"]
    dem = model(case["code"], d)
    L, M, T = settings(case, d)
    sched = case.get("schedule", "serial")
    perms = permutations(dem.m if sched == "layered" else dem.n, L, 2025 + d)
    return P.Graph.from_dem(dem, perms, L=L, M=M, T_max=T, alpha=0.625, lsd_order=case.get("order", 0),
                            message_bits=case.get("bits", 32), schedule=sched)


def pack(s):
    shots, m = s.shape
    wide = torch.zeros((shots, (m + 63) // 64 * 64), dtype=torch.int64, device=s.device)
    wide[:, :m] = s.to(torch.int64)
    bit = torch.ones(64, dtype=torch.int64, device=s.device) << torch.arange(64, device=s.device)
    return (wide.view(shots, -1, 64) * bit).sum(-1)


def prepare(case, seed):
    path, code, d, shots = case["path"], case["code"], case["d"], case["shots"]
    state = {"path": path}
    if path == "ragged":
        ds = [5, 7, 9, 11][: (d - 3) // 2]
        state["pairs"] = [(graph(case, x), syndromes(code, x, shots, seed)) for x in ds]
        state["runtime"] = P.Runtime()
        return state
    state["graph"] = graph(case)
    s = syndromes(code, d, shots, seed)
    state["syndromes"] = pack(s) if path == "packed" else s
    dem = model(code, d)
    if path == "lsd":
        # soft values as the ensemble average leaves them: the channel LLRs,
        # moved by what the members learned from the syndrome
        gen = torch.Generator(device="cuda").manual_seed(seed + 7)
        lam = torch.from_numpy(np.log((1.0 - dem.priors) / dem.priors).astype(np.float32)).cuda()
        state["soft"] = lam + 3.0 * torch.randn((shots, dem.n), generator=gen, device="cuda")
    if path == "grad":
        lam = np.log((1.0 - dem.priors) / dem.priors)
        state["lam"] = torch.from_numpy(lam.astype(np.float32)).cuda()
        state["alpha"] = torch.full((case["K"],), 0.625, device="cuda")
    return state


def run(state):
    path = state["path"]
    if path == "ragged":
        outs = state["runtime"].decode(state["pairs"])
        return [record(*o) for o in outs]
    g, s = state["graph"], state["syndromes"]
    if path == "decode":
        return record(*g.decode(s))
    if path == "packed":
        return record(*g.decode_packed(s))
    if path == "ensemble":
        t_conv, post, ehat = g.bp_ensemble(s)
        return {"t_conv": t_conv, "posteriors": post, "ehat": ehat}
    if path == "lsd":
        corr, stats = g.lsd(s, state["soft"])
        return {"corrections": corr, "stats": stats}
    loss, dlam, dalpha = g.bp_grad(s, state["lam"], state["alpha"])
    return {"loss": loss, "dlam": dlam, "dalpha": dalpha}


def record(corr, obs, stats):
    """Corrections, observables and the fields of the per-shot records that
    the inputs determine (views: nothing is copied)."""
    return {"corrections": corr, "observables": obs, "outcome": stats[:, :3], "lsd": stats[:, 4:7]}


def work(case):
    """Inputs and the graph read once, outputs written once, and the message
    updates of the iterations that the members run: per edge-update a minimum
    and a sign over the row, the scaling, and two sums over the column (6
    operations; the gradient's reverse pass as many again)."""
    path, code, shots = case["path"], case["code"], case["shots"]
    total = 0.0
    ds = [5, 7, 9, 11][: (case["d"] - 3) // 2] if path == "ragged" else [case["d"]]
    for d in ds:
        dem = model(code, d)
        L = settings(case, d)[0]
        words, fb = (dem.n + 63) // 64, 8 if case.get("bits") == 64 else 4
        total += 8.0 * dem.nnz + 8.0 * dem.n + 4.0 * L * dem.n  # H, LLRs, member orders
        total += shots * (dem.m / 8.0 if path == "packed" else dem.m)
        if path == "ensemble":
            total += float(shots) * L * (4 + fb * dem.n + 8 * words)
        elif path == "grad":
            total += 16.0 * dem.n
        else:
            total += shots * (8.0 * words + 33.0) + (4.0 * shots * dem.n if path == "lsd" else 0.0)
    return {"bytes": total, "flops": edge_updates(case) * (12.0 if path == "grad" else 6.0)}


# ------------------------------------------------- the members in 64 bits


def exact(case, seed):
    """The members' posteriors by serial min-sum in 64 bits, every member one
    column at a time in its order.  Corrections and counts are whole numbers,
    which have no value between; the gradient of all shots and members would
    take minutes."""
    if case["path"] != "ensemble":
        return None
    dem = model(case["code"], case["d"])
    L, _, T = settings(case)
    B = case["shots"]
    if dem.n * T > 50000 or B * L * dem.nnz > 3e7:
        return None
    dev, f8 = "cuda", torch.float64
    al, lim, m, n = 0.625, 1e6, dem.m, dem.n
    cols = dem.column_lists()
    D = max(len(c) for c in cols)
    ck = np.full((n, D), m, dtype=np.int64)  # row m: no check
    for v, c in enumerate(cols):
        ck[v, :len(c)] = c
    perm = torch.from_numpy(permutations(n, L, 2025 + case["d"]).astype(np.int64)).to(dev)
    rows = torch.from_numpy(ck).to(dev)[perm]  # [L, n, D]
    real = (rows < m).to(f8)
    lam = torch.from_numpy(np.log((1.0 - dem.priors) / dem.priors)).to(dev)[perm]  # [L, n]
    s = syndromes(case["code"], case["d"], B, seed).to(f8)
    sgn = torch.cat([1.0 - 2.0 * s, torch.ones((B, 1), device=dev, dtype=f8)], 1)  # [B, m + 1]
    idx = [rows[:, a].unsqueeze(1).expand(L, B, D).contiguous() for a in range(n)]
    mu = (lam.unsqueeze(1).unsqueeze(-1) * real.unsqueeze(1)).permute(2, 0, 1, 3).expand(n, L, B, D).contiguous()
    post = torch.empty((L, B, n), device=dev, dtype=f8)
    keep, t_conv = torch.empty_like(post), torch.zeros((L, B), device=dev, dtype=torch.int64)
    h, _ = dense(case["code"], case["d"])
    top = torch.full((L, B, m + 1), lim, device=dev, dtype=f8)
    plus = sgn.unsqueeze(0).expand(L, B, m + 1).contiguous()
    for t in range(1, T + 1):
        # over a row: the least magnitude and the sign of the messages that
        # are still the previous sweep's, after each of its edges
        low, par = top.clone(), torch.ones_like(top)
        later = [None] * n
        for a in range(n - 1, -1, -1):
            q, p = low.gather(2, idx[a]), par.gather(2, idx[a])
            later[a] = (q, p)
            low.scatter_(2, idx[a], torch.minimum(q, mu[a].abs()))
            par.scatter_(2, idx[a], torch.where(mu[a] < 0, -p, p))
        low, par = top.clone(), plus.clone()
        for a in range(n):
            q, p = low.gather(2, idx[a]), par.gather(2, idx[a])
            r = al * torch.minimum(q, later[a][0]) * p * later[a][1] * real[:, a].unsqueeze(1)
            total = lam[:, a].unsqueeze(1) + r.sum(-1)
            post[:, :, a] = total.clamp(-lim, lim)
            others = torch.stack([lam[:, a].unsqueeze(1) + sum(r[..., k] for k in range(D) if k != j) for j in range(D)], -1)
            mu[a] = others.clamp(-lim, lim)
            low.scatter_(2, idx[a], torch.minimum(q, mu[a].abs()))
            par.scatter_(2, idx[a], torch.where(mu[a] < 0, -p, p))
        # a member that converged keeps what it had
        by_col = torch.empty_like(post).scatter_(2, perm.unsqueeze(1).expand(L, B, n), post)
        open_ = t_conv == 0
        keep[open_] = by_col[open_]
        met = (torch.remainder(torch.matmul((by_col <= 0).float(), h), 2.0).round() == s.float()).all(-1)
        t_conv[open_ & met] = t
        if bool((t_conv > 0).all()):
            break
    return {"t_conv": None, "posteriors": keep.permute(1, 0, 2).contiguous(), "ehat": None}
