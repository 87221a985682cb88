"""Performance cases of the assignment-preprocessing path.

Every case goes through the public binding (`paper_1104_3830_amd.Context`) and
stands for one way the library is used: whole solves of one matrix, scaling
alone with each storage and method, batches of ragged instances, real-valued
weights (the paper's Algorithm 1), and the served queue. Sizes and parameters
are those of the benchmark and the tests; `draw` spreads over the same ranges.

A case is a dict of plain values:
  kind      solve | scale | batch | real_solve | real_scale | served
  n, count  matrix size; number of instances (batch, served), whose sizes are
            log-uniform in [lo, hi] and depend on the case alone
  weights   plain (0..100), uniform (0..1000), planted (0..1000 with a
            permutation of weights around 1050), dominant (5% pattern with a
            heavy diagonal); real: random (log of a uniform matrix), euclidean
  stages    length of the ladder 1, 2, 4, ... (real: 100, 150, ...)
  cap       iteration cap per stage (a stage that does not converge by then
            hands its scalings on, as in the benchmark)
  storage, fused, method   options of the scaling
"""
import math
import random
import time

import numpy as np
import torch

import paper_1104_3830_amd as sk

SENTINEL = -32768


def listed():
    return [
        # one small assignment, the n = 64 configuration: latency and launches
        dict(name="solve_plain_64", kind="solve", n=64, weights="plain", stages=4, cap=2000,
             storage="i16", fused=False, method="sinkhorn"),
        # an ordinary instance of odd size whose stages run to the cap
        dict(name="solve_uniform_1003", kind="solve", n=1003, weights="uniform", stages=6, cap=60,
             storage="i16", fused=False, method="sinkhorn"),
        # an ordinary instance that converges at once: the fixed cost of a solve
        dict(name="solve_planted_4096", kind="solve", n=4096, weights="planted", stages=6, cap=60,
             storage="i16", fused=False, method="sinkhorn"),
        # the headline configuration
        dict(name="solve_uniform_16384", kind="solve", n=16384, weights="uniform", stages=6, cap=60,
             storage="i16", fused=False, method="sinkhorn"),
        # the same with one read of the matrix per iteration, a size down
        dict(name="solve_fused_8192", kind="solve", n=8192, weights="uniform", stages=6, cap=60,
             storage="i16", fused=True, method="sinkhorn"),
        # the largest matrices: scaling alone, column entries outside LDS
        dict(name="scale_uniform_32768", kind="scale", n=32768, weights="uniform", stages=6, cap=60,
             storage="i16", fused=False, method="sinkhorn"),
        # stored BF16 K at the size of the planted configuration
        dict(name="scale_bf16_4096", kind="scale", n=4096, weights="uniform", stages=6, cap=60,
             storage="bf16", fused=False, method="sinkhorn"),
        # 512 ragged instances in one call, every stage to its cap
        dict(name="batch_uniform_512", kind="batch", count=512, lo=32, hi=1024, weights="uniform",
             stages=6, cap=100),
        # the same sizes converging at once
        dict(name="batch_planted_512", kind="batch", count=512, lo=32, hi=1024, weights="planted",
             stages=6, cap=500),
        # Algorithm 1 with the paper's defaults on its Euclidean matrix
        dict(name="algorithm1_euclidean_1000", kind="real_solve", n=1000, weights="euclidean"),
        # scaling of a large real-valued matrix
        dict(name="scale_real_8192", kind="real_scale", n=8192, weights="euclidean", stages=2, cap=40),
        # a burst of requests through the served queue
        dict(name="served_64", kind="served", count=64, lo=64, hi=4096, weights="planted", stages=6,
             cap=2000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "scale", "scale", "batch", "batch", "real_solve",
                       "real_scale", "served"])
    if kind == "solve":
        n = _log(rng, 48, 16384)
        fused = n >= 256 and rng.random() < 0.2
        if fused:
            n &= ~7
        weights = rng.choice(["plain", "uniform", "planted", "dominant"])
        return dict(kind=kind, n=n, weights=weights, stages=rng.randint(3, 6),
                    cap=_log(rng, 40, 2000 if n <= 256 else 100), storage="i16", fused=fused,
                    method="sinkhorn")
    if kind == "scale":
        n = _log(rng, 48, 16384)
        storage = rng.choice(["i16", "bf16", "f32"])
        method = "newton" if storage == "i16" and rng.random() < 0.25 else "sinkhorn"
        fused = n >= 256 and method == "sinkhorn" and rng.random() < 0.25
        if fused:
            n &= ~7
        return dict(kind=kind, n=n, weights=rng.choice(["uniform", "planted"]),
                    stages=rng.randint(2, 6) if method == "sinkhorn" else 2, cap=_log(rng, 30, 120),
                    storage=storage, fused=fused, method=method)
    if kind == "batch":
        lo = _log(rng, 32, 256)
        return dict(kind=kind, count=_log(rng, 8, 512), lo=lo, hi=_log(rng, lo + 1, 1024),
                    weights=rng.choice(["uniform", "planted"]), stages=rng.randint(3, 6),
                    cap=_log(rng, 20, 100))
    if kind == "real_solve":
        return dict(kind=kind, n=_log(rng, 200, 2000), weights=rng.choice(["random", "euclidean"]))
    if kind == "real_scale":
        return dict(kind=kind, n=_log(rng, 64, 8192), weights=rng.choice(["random", "euclidean"]),
                    stages=rng.randint(1, 3), cap=_log(rng, 20, 60))
    lo = _log(rng, 64, 512)
    return dict(kind="served", count=_log(rng, 8, 64), lo=lo, hi=_log(rng, lo + 1, 4096),
                weights="planted", stages=6, cap=2000)


# ------------------------------------------------------------------ inputs

def _sizes(case):
    r = random.Random("%d %d %d" % (case["count"], case["lo"], case["hi"]))
    return [_log(r, case["lo"], case["hi"]) for _ in range(case["count"])]


def _ladder(case):
    if case["kind"].startswith("real"):
        return [100 + 50 * k for k in range(case["stages"])]
    return [1 << k for k in range(case["stages"])]


def _weights(n, weights, g):
    """int16 log-weights (n, n) on the device."""
    hi = 100 if weights == "plain" else 600 if weights == "dominant" else 1000
    W = torch.randint(0, hi + 1, (n, n), generator=g, device="cuda", dtype=torch.int16)
    if weights == "planted":
        sigma = torch.randperm(n, generator=g, device="cuda")
        W[torch.arange(n, device="cuda"), sigma] = torch.randint(
            1040, 1061, (n,), generator=g, device="cuda", dtype=torch.int16)
    elif weights == "dominant":
        for r in range(0, n, 2048):
            part = W[r:r + 2048]
            part[torch.rand(part.shape, generator=g, device="cuda") >= 0.05] = SENTINEL
        W.diagonal().copy_(torch.randint(800, 1001, (n,), generator=g, device="cuda",
                                         dtype=torch.int16))
    return W


def _real_weights(n, weights, g):
    """float32 log-weights (n, n) on the device."""
    if weights == "random":
        return torch.log1p(-torch.rand((n, n), generator=g, device="cuda"))
    x = torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)
    y = torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)
    W = torch.empty((n, n), device="cuda")
    for r in range(0, n, 1024):
        d = x[r:r + 1024, None, :] - y[None, :, :]
        W[r:r + 1024] = -d.square().sum(2).sqrt()
    return W


def _generator(seed):
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    return g


def _inputs(case, seed):
    g = _generator(seed)
    if case["kind"] in ("batch", "served"):
        return [_weights(n, case["weights"], g) for n in _sizes(case)]
    if case["kind"].startswith("real"):
        return _real_weights(case["n"], case["weights"], g)
    return _weights(case["n"], case["weights"], g)


def _params(case):
    n, kind = case.get("n"), case["kind"]
    if kind == "real_solve":
        return sk.paper_params(n)
    if kind == "real_scale":
        return sk.make_params(_ladder(case), tol=1.0 / n, max_iters=case["cap"], threshold=1.0 / n,
                              prescale=True)
    return sk.make_params(_ladder(case), tol=1e-5, max_iters=case["cap"], threshold=1e-4,
                          storage=case.get("storage", "i16"), fused=case.get("fused", False),
                          method=case.get("method", "sinkhorn"))


def prepare(case, seed):
    kind = case["kind"]
    prm = _params(case)
    W = _inputs(case, seed)
    state = dict(kind=kind, params=prm)
    if kind == "served":
        state["W"] = [w.cpu().numpy() for w in W]
        state["ctx"] = sk.Context(0, arena_bytes=1 << 30)
        # the queue's threads and staging are up before requests arrive
        n = case["lo"]
        _served(state["ctx"], [np.zeros((n, n), np.int16)], prm)
        return state
    state["W"] = W
    if kind == "batch":
        # the potentials of all instances in one buffer, instance k's four
        # arrays of n behind one another from 16 * off[k] on
        sizes = _sizes(case)
        flat = torch.zeros(16 * sum(sizes), dtype=torch.uint8, device="cuda")
        at, pots, iu = 0, [], []
        for n in sizes:
            pots.append(flat[16 * at:16 * (at + n)])
            iu.append(torch.arange(4 * at, 4 * at + n))
            at += n
        ns = torch.tensor(sizes)
        state.update(flat=flat, pots=pots, iu=torch.cat(iu).cuda(),
                     n_of=torch.repeat_interleave(ns, ns).cuda())
        state["ctx"] = sk.Context(0, arena_bytes=256 << 20)
    else:
        n = case["n"]
        state["pot"] = torch.zeros(sk.potentials_bytes(n), dtype=torch.uint8, device="cuda")
        if kind == "real_solve":
            need = int(sk.lib().sk_real_arena_bytes(n, n * n))
        elif kind == "real_scale":
            need = int(sk.lib().sk_real_arena_bytes(n, 0))
        elif kind == "scale":
            need = int(sk.lib().sk_arena_bytes(n, prm.storage))
        else:
            need = int(sk.lib().sk_solve_arena_bytes(n, prm.storage, 64 * n + 4096))
        state["ctx"] = sk.Context(0, arena_bytes=need)
    return state


# ------------------------------------------------------------------ one pass

def _logs(pot):
    """(log u, log v) on the device from a potentials buffer (F, phi, G, gam)."""
    i, f = pot.view(torch.int32).view(4, -1), pot.view(torch.float32).view(4, -1)
    return i[0] + f[1], i[2] + f[3]


def _served(ctx, Ws, prm):
    out, tickets, nxt = [None] * len(Ws), {}, 0
    while nxt < len(Ws) or tickets:
        while nxt < len(Ws):
            try:
                tickets[ctx.submit(Ws[nxt], prm)] = nxt
            except sk.SkError as e:
                if e.status != sk.SK_EAGAIN:
                    raise
                break
            nxt += 1
        done = ctx.completed()
        for t in done:
            k = tickets.pop(t)
            out[k] = ctx.poll(t, Ws[k].shape[0])
        if not done:
            time.sleep(2e-5)
    return out


def run(state):
    kind, ctx, prm, W = state["kind"], state["ctx"], state["params"], state["W"]
    if kind == "served":
        got = _served(ctx, W, prm)
        return dict(perm=np.concatenate([g[1] for g in got]), weight=np.array([g[2] for g in got]))
    if kind == "batch":
        ctx.scale_batch(W, prm, potentials=state["pots"])
        i, f = state["flat"].view(torch.int32), state["flat"].view(torch.float32)
        iu, n = state["iu"], state["n_of"]
        return dict(log_u=i[iu] + f[iu + n], log_v=i[iu + 2 * n] + f[iu + 3 * n])
    if kind == "scale":
        ctx.scale(W, prm, potentials=state["pot"])
    elif kind == "real_scale":
        ctx.scale_real(W, prm, potentials=state["pot"])
    else:
        solve = ctx.solve_real if kind == "real_solve" else ctx.solve
        out = solve(W, prm, potentials=state["pot"])
        log_u, log_v = _logs(state["pot"])
        weight = out["weight"] if kind == "solve" else np.float32(out["weight"])
        return dict(perm=out["perm"], weight=weight, ub=np.float32(out["report"]["ub"]),
                    log_u=log_u, log_v=log_v)
    log_u, log_v = _logs(state["pot"])
    return dict(log_u=log_u, log_v=log_v)


def work(case):
    """Bytes: the matrix read once, potentials and assignment written once.
    Flops: a multiply-add per entry and sweep, one iteration per stage."""
    kind = case["kind"]
    sizes = _sizes(case) if "count" in case else [case["n"]]
    elem = 4 if kind.startswith("real") else 2
    squares = sum(n * n for n in sizes)
    out = 16 if kind != "served" else 0
    if kind in ("solve", "real_solve", "served"):
        out += 4
    return dict(bytes=elem * squares + out * sum(sizes), flops=4 * squares * case.get("stages", 1))


# ------------------------------------------------------------------ in 64 bits

def _scalings(W, ladder, tol, cap):
    """log u, log v of the Sinkhorn iteration with continuation, in float64:
    W (batch, n, m) float64, -inf for a zero entry; rows or columns that are
    all -inf are padding. Each instance of the batch stops by itself."""
    rows = (W > -math.inf).any(2)
    cols = (W > -math.inf).any(1)
    f = torch.where(rows, -ladder[0] * W.amax(2), 0.0)
    g = torch.zeros(cols.shape, dtype=torch.float64, device=W.device)
    for s, p in enumerate(ladder):
        if s:
            f, g = f * (p / ladder[s - 1]), g * (p / ladder[s - 1])
        K = W * p
        K += f[:, :, None]
        K += g[:, None, :]
        K.exp_()
        a, b = rows.double(), cols.double()
        live = torch.ones(W.shape[0], dtype=torch.bool, device=W.device)
        for it in range(cap):
            S = torch.matmul(K, b[:, :, None])[:, :, 0]
            if it and tol > 0:
                res = torch.where(rows, (a * S - 1).abs(), 0.0).amax(1)
                live = live & ~(res < tol)
                if not bool(live.any()):
                    break
            a2 = torch.where(rows, 1 / S, 0.0)
            T = torch.matmul(a2[:, None, :], K)[:, 0, :]
            b2 = torch.where(cols, 1 / T, 0.0)
            a = torch.where(live[:, None], a2, a)
            b = torch.where(live[:, None], b2, b)
        del K
        f = f + torch.where(rows, a, 1.0).log()
        g = g + torch.where(cols, b, 1.0).log()
    return f, g


def _wide(w):
    W = w.double()
    return W.masked_fill_(w == SENTINEL, -math.inf) if w.dtype == torch.int16 else W


def _certificate(W, p, g):
    """The bound of the optimal assignment's weight from the column scalings."""
    return float(((p * W + g).amax(1).sum() - g.sum()) / p)


def exact(case, seed):
    kind = case["kind"]
    if kind == "served":  # whole numbers only
        return None
    if kind == "real_solve":  # the last stage depends on the assignments found on the way
        return None
    if case.get("method") == "newton":  # unique up to a scalar only
        return None
    tol = float(np.float32(1.0 / case["n"] if kind == "real_scale" else 1e-5))
    inputs = _inputs(case, seed)
    if kind == "batch":
        # instances of a size class together, padded to its largest
        sizes = _sizes(case)
        log_u, log_v = [None] * len(sizes), [None] * len(sizes)
        classes = {}
        for k, n in enumerate(sizes):
            classes.setdefault(int(4 * math.log2(n)), []).append(k)
        for ks in classes.values():
            m = max(sizes[k] for k in ks)
            W = torch.full((len(ks), m, m), -math.inf, dtype=torch.float64, device="cuda")
            for q, k in enumerate(ks):
                W[q, :sizes[k], :sizes[k]] = _wide(inputs[k])
            f, g = _scalings(W, _ladder(case), tol, case["cap"])
            for q, k in enumerate(ks):
                log_u[k], log_v[k] = f[q, :sizes[k]], g[q, :sizes[k]]
        return dict(log_u=torch.cat(log_u), log_v=torch.cat(log_v))
    W = _wide(inputs)
    del inputs
    ladder = [float(p) for p in _ladder(case)]
    if kind == "real_scale":
        top, low = float(W.max()), float(W.min())
        W -= top
        if top - low > 1:
            ladder = [p / (top - low) for p in ladder]
    f, g = _scalings(W[None], ladder, tol, case["cap"])
    out = dict(log_u=f[0], log_v=g[0])
    if kind == "solve":
        out.update(perm=None, weight=None, ub=_certificate(W, ladder[-1], g[0]))
    return out
