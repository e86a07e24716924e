"""The measured calls of this framework: what a program that solves knapsack
allocations with it does, through the package's public entry points.

listed() are fixed cases, draw(rng) gives more of the same ranges, prepare()
makes the inputs and the handles such a program keeps, run() is one pass,
work() what a pass cannot do without, exact() the same results in plain torch
in 64 bits.

A case's keys: `call` (the entry point), N users, M items, K knapsacks, `costs`
("dense", "pairs": two knapsacks per item in rows of equal length, "ragged":
0..4 knapsacks per item), `sets` ("top": one cap Q, "halves": a cap of 3 over
two halves capped at 2, "nested": four groups capped at Q under a cap of 2 Q,
"copies": every item may be taken twice, Q in all), `profits`, `share` (a budget
as a share of the total demand), `start` ("zero", "near": the multipliers of a
small sample, "low": U(0, 1/K)) and `steps` (iterations of one pass).
"""
import math

import numpy as np
import torch

import paper_2002_00352_amd as kp

DEV = "cuda"


def _case(name, call, N, M, K, Q, **kw):
    c = dict(call=call, N=N, M=M, K=K, Q=Q, costs="dense", sets="top", profits="uniform", share=0.02,
             start="zero", steps=1)
    c.update(kw)
    return dict(c, name=name)


def listed():
    return [
        # a request-sized dual evaluation with its decisions: latency and launches count
        _case("dual_small", "dual", 10_000, 10, 2, 1, start="low"),
        # the whole solve of a small instance, sweeps, gap checks and post-processing included
        _case("solve_small", "solve", 10_000, 10, 2, 1, steps=20),
        # dual descent on a mid-sized dense instance
        _case("descent_dense", "descent", 3_000_000, 10, 10, 3, profits="lognormal", share=0.01, start="low", steps=3),
        # the dual and its gradient through autograd, long rows of costs
        _case("grad_wide", "grad", 500_000, 20, 50, 5, share=0.005, start="low"),
        # coordinate descent from zero on dense costs (densely coupled knapsacks)
        _case("scd_dense", "scd", 1_000_000, 10, 10, 3, profits="lognormal", share=0.01, steps=4),
        # the same with long rows
        _case("scd_wide", "scd", 200_001, 20, 50, 5, share=0.005, steps=4),
        # the hierarchical sparse workload from zero: the cold start of a solve
        _case("scd_pairs_cold", "scd", 5_000_000, 10, 20, 3, costs="pairs", sets="halves", profits="exp", share=0.05, steps=4),
        # the same at scale from a pre-solved start: the steady iterations, the largest case
        _case("scd_pairs_near", "scd", 20_000_000, 10, 20, 3, costs="pairs", sets="halves", profits="exp", share=0.05,
              start="near", steps=4),
        # a feasible answer at the end of a solve: post-processing with its decisions
        _case("fixup_pairs", "fixup", 10_000_000, 10, 20, 3, costs="pairs", sets="halves", profits="exp", share=0.05, start="near"),
        # item rows of unequal length, an odd item count, nested sets
        _case("scd_ragged", "scd", 300_007, 23, 12, 2, costs="ragged", sets="nested", profits="exp", share=0.05, steps=4),
        # categorical variables: every item up to twice, as binary copies
        _case("scd_copies", "scd", 500_000, 20, 20, 3, costs="pairs", sets="copies", profits="exp", share=0.05, steps=4),
        # many ragged instances iterated together
        _case("batched", "batched", 100_000, 32, 16, 4, share=0.1, steps=4),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["dual", "solve", "descent", "grad", "scd", "scd", "scd", "scd", "fixup", "batched"])
    M, K, Q = rng.randint(4, 32), rng.randint(2, 32), rng.randint(1, 5)
    c = dict(call=call, M=M, K=K, Q=Q, sets="top", profits=rng.choice(["uniform", "exp", "lognormal"]), steps=1)
    c["costs"] = "dense" if call in ("batched", "grad") else rng.choice(["dense", "pairs", "ragged"])
    if call in ("scd", "dual", "fixup"):
        c["sets"] = rng.choice(["top", "halves", "nested"] + (["copies"] if c["costs"] == "pairs" else []))
    if c["sets"] == "copies":
        c["M"] = M = M // 2 * 2
    c["share"] = rng.choice([0.2, 0.4, 0.8]) * min(Q, M) / M / (1 if c["costs"] != "dense" else 2)
    c["start"] = {"solve": "zero", "batched": "zero", "fixup": "near", "scd": rng.choice(["zero", "near"])}.get(call, "low")
    c["steps"] = {"solve": 20, "descent": 3, "scd": 4, "batched": 4}.get(call, 1)
    # bytes of one pass over p and b, at most what a listed case of that call has
    row = M * (4 + {"dense": 4 * K, "pairs": 16, "ragged": 32}[c["costs"]])
    top = {"dual": 4e8, "solve": 2e7, "descent": 1e9, "grad": 2e9, "scd": 4e8, "fixup": 1e9, "batched": 1e9}[call]
    c["N"] = _spread(rng, 1000, max(2000, int(top / row))) if call != "batched" else _spread(rng, 5000, 60000)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sets(c):
    """Local sets as lists of (items, cap), subsets first."""
    M, Q = c["M"], c["Q"]
    every = list(range(M))
    if c["sets"] == "top":
        return [(every, Q)]
    if c["sets"] == "halves":
        return [(every[:M // 2], 2), (every[M // 2:], 2), (every, 3)]
    if c["sets"] == "nested":
        w = -(-M // 4)
        return [(every[i:i + w], Q) for i in range(0, M, w)] + [(every, 2 * Q)]
    return [(every[i:i + 2], 2) for i in range(0, M, 2)] + [(every, Q)]  # copies


def _rand(gen, n):
    return torch.rand(n, generator=gen, device=DEV, dtype=torch.float32)  # on a grid of 2^-24


def _profits(kind, gen, n):
    if kind == "lognormal":
        return torch.empty(n, device=DEV).log_normal_(0.0, 1.0, generator=gen)
    u = _rand(gen, n)
    return u if kind == "uniform" else -torch.log1p(-u)


def _arrays(c, seed, N=None, M=None, K=None):
    """p, and b or (rowptr, col, val), and the budgets' total demand."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    N, M, K = N or c["N"], M or c["M"], K or c["K"]
    copies = 2 if c["sets"] == "copies" else 1
    rows = N * M // copies
    d = dict(p=_profits(c["profits"], gen, rows))
    if c["costs"] == "dense":
        d["b"] = _rand(gen, rows * K)
        D = d["b"].view(-1, K).sum(0, dtype=torch.float64)
    elif c["costs"] == "pairs":
        a = torch.randint(0, K, (rows,), generator=gen, device=DEV, dtype=torch.int32)
        b = torch.randint(0, K - 1, (rows,), generator=gen, device=DEV, dtype=torch.int32)
        b += (b >= a).to(torch.int32)
        d["col"] = torch.stack((torch.minimum(a, b), torch.maximum(a, b)), 1).reshape(-1)
        d["val"] = _rand(gen, rows * 2)
    else:
        # every (item, knapsack) entry with chance 2/K, at most 4 an item
        keep = torch.rand((rows, K), generator=gen, device=DEV) < min(1.0, 2.0 / K)
        keep &= torch.cumsum(keep.to(torch.uint8), 1, dtype=torch.uint8) <= 4
        d["col"] = keep.nonzero()[:, 1].to(torch.int32).contiguous()
        d["rowptr"] = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(keep.sum(1), 0, out=d["rowptr"][1:])
        d["val"] = _rand(gen, d["col"].numel())
    if copies == 2:  # the two copies of an item share its profit and its entries
        d["p"] = d["p"].repeat_interleave(2)
        for k in ("col", "val"):
            d[k] = d[k].view(rows, 1, 2).expand(rows, 2, 2).reshape(-1).contiguous()
    if c["costs"] != "dense":
        if "rowptr" not in d:
            d["rowptr"] = torch.arange(N * M + 1, dtype=torch.int64, device=DEV) * 2
        D = torch.stack([torch.where(d["col"] == k, d["val"], 0.0).sum(dtype=torch.float64) for k in range(K)])
    return d, np.maximum(D.cpu().numpy() * c["share"], 1e-3)


def _batch(c, seed):
    """Shapes of the batch's instances: N spread over two decades, ragged M, K and Q."""
    r = np.random.RandomState(c["N"])
    out = []
    for i in range(32):
        one = dict(c, N=int(c["N"] * 10 ** -r.uniform(0, 2)) + 1, M=int(r.randint(4, c["M"] + 1)),
                   K=int(r.randint(1, c["K"] + 1)), Q=int(r.randint(1, c["Q"] + 1)))
        out.append((one, (seed * 1009 + i) % (1 << 31)))
    return out


def _problem(c, d, B):
    sets = _sets(c)
    parent, cap, leaf = kp.kp_tree_from_sets(c["M"], [s for s, _ in sets], [q for _, q in sets])
    return kp.Problem(d["p"], B, parent, cap, leaf, N=c["N"], M=c["M"], K=c["K"],
                      **{k: v for k, v in d.items() if k != "p"})


def _start(c, seed, d, B):
    K = c["K"]
    if c["start"] == "zero":
        return torch.zeros(K, dtype=torch.float64, device=DEV)
    if c["start"] == "low":
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed + 1)
        return torch.rand(K, generator=gen, device=DEV, dtype=torch.float64) / K
    # the multipliers of a sample after a few sweeps, every knapsack bisected at once
    n = min(c["N"], 1000)
    P, C = _dense(c, d, 0, n)
    b = C.permute(2, 0, 1).contiguous()
    Bs = torch.from_numpy(B * (n / c["N"])).to(DEV)
    lam = torch.zeros(K, dtype=torch.float64, device=DEV)
    for _ in range(4):
        z0 = _scored(P, C, lam) + lam[:, None, None] * b
        lo, hi = torch.zeros_like(lam), torch.where(b > 0, z0 / b, 0.0).amax((1, 2)).clamp(min=1e-3)
        for _ in range(30):
            mid = 0.5 * (lo + hi)
            over = (_greedy(c, z0 - mid[:, None, None] * b) * b).sum((1, 2)) > Bs
            lo, hi = torch.where(over, mid, lo), torch.where(over, hi, mid)
        lam = torch.where(hi < 1e-6, 0.0, hi)
    return lam


def prepare(case, seed):
    c = case
    if c["call"] == "batched":
        probs = []
        for one, s in _batch(c, seed):
            d, B = _arrays(one, s)
            probs.append(_problem(one, d, B))
        return dict(c=c, plan=kp.BatchedSCD(probs))
    d, B = _arrays(c, seed)
    s = dict(c=c, prob=_problem(c, d, B), lam=_start(c, seed, d, B), ctx=kp.Context())
    s["alpha"] = 10.0 / c["N"]
    return s


def run(state):
    c = state["c"]
    if c["call"] == "batched":
        plan = state["plan"]
        with torch.cuda.stream(plan.stream):
            torch._foreach_zero_(plan.lam)
            for _ in range(c["steps"]):
                lam, stats = plan.step()
        return dict(lam=lam, stats=stats)
    prob, lam, ctx = state["prob"], state["lam"], state["ctx"]
    if c["call"] == "dual":
        return kp.kp_eval_dual(prob, lam, want_x=True, ctx=ctx)
    if c["call"] == "grad":
        lam = lam.clone().requires_grad_(True)
        g = kp.DualFn.apply(lam, prob)
        g.backward()
        return dict(g=g.detach(), grad=lam.grad)
    if c["call"] == "descent":
        lam = lam.clone()
        for _ in range(c["steps"]):
            out = kp.kp_dd_step(prob, state["alpha"], lam, ctx=ctx)
        return out
    if c["call"] == "scd":
        for _ in range(c["steps"]):
            out = kp.kp_scd_sweep(prob, lam, ctx=ctx)
            lam = out["lam"]
        return out
    if c["call"] == "fixup":
        return kp.kp_primal_fixup(prob, lam, want_x=True, ctx=ctx)
    lam, hist = kp.solve(prob, "scd", tol=1e-3, max_iter=c["steps"])
    return dict(lam=lam, g=[h["g"] for h in hist], P=[h["P"] for h in hist], best=[h["best_P"] for h in hist])


def work(case):
    """p and b once per step, and the decisions where they are returned; a multiplication and an addition per cost entry."""
    def once(c):
        ent = c["N"] * c["M"] * {"dense": c["K"], "pairs": 2, "ragged": min(2, c["K"])}[c["costs"]]
        return c["N"] * c["M"] * 4 + ent * (4 if c["costs"] == "dense" else 8), 2.0 * ent
    c = case
    if c["call"] == "batched":
        by, fl = (sum(v) for v in zip(*(once(one) for one, _ in _batch(c, 0))))
    else:
        by, fl = once(c)
    steps = 8 if c["call"] == "solve" else c["steps"]  # a small solve takes about 8 sweeps
    x = c["N"] * c["M"] if c["call"] in ("dual", "fixup") else 0
    return {"bytes": float(by * steps + x), "flops": fl * steps}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _dense(c, d, i0, i1):
    """Profits [n, M] and costs [n, M, K] of the users i0..i1 in 64 bits."""
    M, K, n = c["M"], c["K"], i1 - i0
    P = d["p"].view(-1, M)[i0:i1].double()
    if "b" in d:
        return P, d["b"].view(-1, M, K)[i0:i1].double()
    e0, e1 = (int(v) for v in d["rowptr"][[i0 * M, i1 * M]])
    ln = d["rowptr"][i0 * M + 1:i1 * M + 1] - d["rowptr"][i0 * M:i1 * M]
    row = torch.repeat_interleave(torch.arange(n * M, device=DEV), ln)
    C = torch.zeros((n * M, K), dtype=torch.float64, device=DEV)
    C[row, d["col"][e0:e1].long()] = d["val"][e0:e1].double()
    return P, C.view(n, M, K)


def _greedy(c, z):
    """The selected items of every user (last axis) at the lines' values z."""
    order = torch.argsort(z, dim=-1, descending=True, stable=True)
    alive = torch.gather(z, -1, order) > 0
    for items, cap in _sets(c):
        inset = torch.zeros(c["M"], dtype=torch.bool, device=DEV)
        inset[items] = True
        m = inset[order] & alive
        alive &= ~(m & (torch.cumsum(m.to(torch.int32), -1) > cap))
    return torch.zeros_like(alive).scatter_(-1, order, alive)


def _scored(P, C, lam):
    z = P.clone()
    for k in range(C.shape[-1]):
        z -= lam[k] * C[..., k]
    return z


def _thresholds(c, parts, lam, B):
    """One synchronous update: per knapsack the largest multiplier at which the consumption still exceeds its budget (0: none),
    by bisection; users whose consumption agrees at both ends keep it in between and leave."""
    out = torch.zeros_like(lam)
    Z = [_scored(P, C, lam) for P, C in parts]
    for k in range(c["K"]):
        b = [C[..., k] for _, C in parts]
        z0 = [z + lam[k] * bk for z, bk in zip(Z, b)]
        def use(zz, bb, at):
            return (_greedy(c, zz - at * bb) * bb).sum(-1)
        tiny = 1e-300
        if sum(float(use(zz, bb, tiny).sum()) for zz, bb in zip(z0, b)) <= B[k]:
            continue
        hi = max(float((zz / bb)[bb > 0].max()) for zz, bb in zip(z0, b) if bool((bb > 0).any()))
        lo, hi, fixed = 0.0, hi * (1 + 1e-12) + tiny, 0.0
        ulo = [use(zz, bb, tiny) for zz, bb in zip(z0, b)]
        uhi = [torch.zeros_like(u) for u in ulo]
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            if not lo < mid < hi:
                break
            um = [use(zz, bb, mid) for zz, bb in zip(z0, b)]
            over = fixed + sum(float(u.sum()) for u in um) > B[k]
            lo, hi = (mid, hi) if over else (lo, mid)
            ulo, uhi = (um, uhi) if over else (ulo, um)
            for i in range(len(b)):
                open_ = ulo[i] != uhi[i]
                fixed += float(uhi[i][~open_].sum())
                z0[i], b[i], ulo[i], uhi[i] = (v[open_] for v in (z0[i], b[i], ulo[i], uhi[i]))
            if not sum(u.numel() for u in ulo):
                break
        out[k] = 0.5 * (lo + hi)
    return out


def _evaluate(c, d, lam, B, keep_x=False):
    M, K = c["M"], c["K"]
    R = torch.zeros(K, dtype=torch.float64, device=DEV)
    g = P_sum = 0.0
    xs = []
    step = max(1, int(2e8 / (M * K * 8)))
    for i0 in range(0, c["N"], step):
        P, C = _dense(c, d, i0, min(c["N"], i0 + step))
        z = _scored(P, C, lam)
        x = _greedy(c, z)
        R += (C * x[..., None]).sum((0, 1))
        g += float((z * x).sum())
        P_sum += float((P * x).sum())
        if keep_x:
            xs.append(x)
    g += float((lam.cpu() * torch.from_numpy(B)).sum())
    return R, torch.tensor([g], dtype=torch.float64), torch.tensor([P_sum], dtype=torch.float64), (torch.cat(xs) if keep_x else None)


def exact(case, seed):
    c = case
    size = c["N"] * c["M"] * c["K"]
    if c["call"] in ("batched", "solve"):
        return None
    if c["call"] == "scd" and size * c["K"] * c["steps"] > 4e10:
        return None
    d, B = _arrays(c, seed)
    lam = _start(c, seed, d, B)
    Bt = torch.from_numpy(B).to(DEV)
    if c["call"] == "scd":
        for _ in range(c["steps"]):
            old = lam
            step = max(1, int(4e9 / (c["M"] * c["K"] * 8)))
            parts = [_dense(c, d, i0, min(c["N"], i0 + step)) for i0 in range(0, c["N"], step)]
            lam = _thresholds(c, parts, old, B)
        R, g, P, _ = _evaluate(c, d, old, B)
        return dict(lam=lam, R=R, g=g, P=P)
    if c["call"] == "descent":
        for _ in range(c["steps"]):
            R, g, P, _ = _evaluate(c, d, lam, B)
            lam = torch.clamp(lam + 10.0 / c["N"] * (R - Bt), min=0)
        return dict(lam=lam, R=R, g=g, P=P)
    R, g, P, x = _evaluate(c, d, lam, B, keep_x=True)
    if c["call"] == "grad":
        return dict(g=g.reshape(()), grad=Bt - R)
    if c["call"] == "dual":
        return dict(R=R, g=g, P=P, x=x.to(torch.uint8).reshape(-1))
    # post-processing: users that consume a violated knapsack leave in the order of their dual value
    over = (R > Bt).nonzero()[:, 0].tolist()
    use, G, worth = [], [], []
    step = max(1, int(2e8 / (c["M"] * c["K"] * 8)))
    for i0 in range(0, c["N"], step):
        Pp, C = _dense(c, d, i0, min(c["N"], i0 + step))
        xx = x[i0:i0 + step]
        use.append((C * xx[..., None]).sum(1))
        G.append((_scored(Pp, C, lam) * xx).sum(-1))
        worth.append((Pp * xx).sum(-1))
    use, G, worth = torch.cat(use), torch.cat(G), torch.cat(worth)
    cand = (use[:, over] > 0).any(1).nonzero()[:, 0] if over else torch.zeros(0, dtype=torch.int64, device=DEV)
    order = cand[torch.argsort(G[cand], stable=True)]
    n = 0
    for k in over:
        left = R[k] - torch.cumsum(use[order, k], 0)
        n = max(n, int((left > Bt[k]).sum()) + 1)
    gone = order[:n]
    x[gone] = False
    return dict(x=x.to(torch.uint8).reshape(-1), P=P.to(DEV) - worth[gone].sum(), R=R - use[gone].sum(0), n_reset=None)
