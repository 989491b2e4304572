"""Performance cases of the FASGD parameter-server library.

Each case is one call (or the pair of calls) that a server makes per arrival,
through the Python binding, at the sizes of this repository's workloads:
100,000 parameters (the tiny trace), 1,796,010 (a 784-1000-1000-10 MLP),
25 million and the memory-scale vector of up to 1e9.  The kinds:

  dense     fasgd_apply_updates / sasgd_apply_updates: K queued client
            gradients in one pass
  step      fasgd_apply_with_push_and_select: the pipelined server step (a
            queued push, K gradients, the next push's selection)
  push      bfasgd_select_compact, then bfasgd_apply_sparse: one B-FASGD push
            from decision to server update
  pushes    bfasgd_select_compact_batch, then fasgd_apply_pushes: B pushes
            that arrive together
  select    bfasgd_select_compact with the list's index: the client side of a
            push on its own
  cached    selection, then bfasgd_apply_cached: a push whose dropped values
            re-apply the client's most recent gradient
  fetch     selection over the server's parameters, then bfasgd_apply_fetch:
            a client refreshes its copy
  segments  bfasgd_decide_segments, then bfasgd_apply_segments: one decision
            per tensor

Inputs follow the workloads' recipe: theta ~ N(0, 0.05^2), gradients
m + s z with m ~ N(0, 1e-3^2), s log-uniform in [1e-4, 1e-1] per parameter
(per tensor for "segments"), and statistics n, b, v as a running server holds
them.  The server starts at a timestamp past every delay.
"""
import math
import random

import numpy as np
import torch

import paper_1601_04033_amd as fa

GAMMA, BETA, EPS = 0.95, 0.9, 1e-4
EPS_C = 1e-8
MLP = (784 * 1000, 1000, 1000 * 1000, 1000, 1000 * 10, 10)   # W1 b1 W2 b2 W3 b3
MLP_P = sum(MLP)
MOST_BYTES = 66e9     # device memory of one state
T0 = 4096             # the server's timestamp before the first pass


def listed():
    return [
        # the smallest server: one gradient per pass over 100k parameters, bound by latency
        {"name": "tiny_fasgd_k1", "kind": "dense", "P": 100_000, "K": 1, "lam": 4, "rule": "fasgd", "math": "fast"},
        # an MLP server with 16 clients whose gradients are applied 16 at a time (P mod 4 = 2)
        {"name": "mlp_fasgd_k16", "kind": "dense", "P": MLP_P, "K": 16, "lam": 16, "rule": "fasgd", "math": "fast"},
        # a 25M-parameter server with a short queue
        {"name": "large_fasgd_k8", "kind": "dense", "P": 25_000_000, "K": 8, "lam": 64, "rule": "fasgd", "math": "fast"},
        # the same server with a full queue and correctly rounded arithmetic
        {"name": "large_fasgd_k32_ieee", "kind": "dense", "P": 25_000_000, "K": 32, "lam": 64, "rule": "fasgd",
         "math": "ieee"},
        # the staleness-aware baseline rule at the same size
        {"name": "large_sasgd_k32", "kind": "dense", "P": 25_000_000, "K": 32, "lam": 64, "rule": "sasgd", "math": "fast"},
        # the memory-scale server's step, as large as three sets of its inputs fit one GPU
        {"name": "memscale_step_k32", "kind": "step", "P": 400_000_000, "K": 32, "lam": 256, "math": "fast", "f": 0.1},
        # one MLP-sized B-FASGD push at 20 % (a 5x bandwidth reduction), decided, compacted and applied
        {"name": "mlp_push", "kind": "push", "P": MLP_P, "lam": 16, "math": "fast", "f": 0.2},
        # the pushes of 16 clients that reach the MLP server together
        {"name": "mlp_pushes_b16", "kind": "pushes", "P": MLP_P, "B": 16, "lam": 16, "math": "fast", "f": 0.2},
        # the selection of a memory-scale push at 10 %
        {"name": "memscale_select", "kind": "select", "P": 1_000_000_000, "lam": 256, "f": 0.1},
        # a 25M push at 10 % whose dropped values re-apply the client's cached gradient
        {"name": "large_cached", "kind": "cached", "P": 25_000_000, "lam": 64, "math": "fast", "f": 0.1},
        # a client's 10 % refresh of its copy of a ragged 100M-parameter vector
        {"name": "ragged_fetch", "kind": "fetch", "P": 99_999_989, "lam": 64, "f": 0.1},
        # the paper's own decision per tensor of the MLP, and its server update (most pushes are sent: the paper
        # finds that dropping even a few hurts)
        {"name": "mlp_segments", "kind": "segments", "P": MLP_P, "S": 6, "lam": 16, "math": "fast", "f": 0.8},
    ]


def _footprint(c):
    """Device bytes of one state of the case."""
    P, kind = c["P"], c["kind"]
    if kind == "dense":
        return P * (20 + 4 * c["K"])
    if kind == "step":
        return P * (20 + 4 * (c["K"] + 1) + 8)
    if kind == "pushes":
        return P * (20 + 12 * c["B"])
    return P * 36


def draw(rng):
    kind = rng.choice(["dense", "dense", "dense", "step", "push", "pushes", "select", "cached", "fetch", "segments"])
    c = {"kind": kind, "lam": rng.choice([1, 4, 16, 64, 256])}
    if kind in ("dense", "step"):
        c["K"] = rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 24, 32])
    if kind == "dense":
        c["rule"] = rng.choice(["fasgd", "fasgd", "fasgd", "sasgd"])
    if kind == "pushes":
        c["B"] = rng.choice([2, 3, 4, 8, 16, 32])
    if kind in ("dense", "step", "push", "pushes", "cached", "segments"):
        c["math"] = rng.choice(["fast", "fast", "fast", "ieee"])
    if kind == "segments":
        c["S"] = rng.choice([1, 6, 16, 50, 100])
        c["f"] = 0.8
    elif kind != "dense":
        c["f"] = rng.choice([0.05, 0.1, 0.2, 0.3])
    c["P"] = 1
    most = min(4e8, MOST_BYTES / _footprint(c), 40e6 if kind in ("pushes", "segments") else 4e8)
    c["P"] = int(math.exp(rng.uniform(math.log(2e4), math.log(most))))
    return c


def _segments(c):
    """Host offsets of the case's tensors (S + 1 of them)."""
    if c["P"] == MLP_P and c["S"] == len(MLP):
        return np.concatenate([[0], np.cumsum(MLP)]).astype(np.int64)
    rng = random.Random(c["P"] * 1009 + c["S"])
    cuts = sorted(rng.sample(range(1, c["P"]), c["S"] - 1))
    return np.array([0] + cuts + [c["P"]], dtype=np.int64)


def _alpha(c):
    return 0.04 if c.get("rule") == "sasgd" else 0.005


def _arrivals(c, seed, count):
    """Clients and delays of `count` arrivals."""
    rng = random.Random(seed * 7919 + 3)
    return [rng.randrange(c["lam"]) for _ in range(count)], [rng.randint(0, 2 * c["lam"]) for _ in range(count)]


def _inputs(c, seed):
    """The case's arrays, from the seed alone."""
    P, kind = c["P"], c["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1_000_003 + 17)

    def normal(scale):
        x = torch.empty(P, device="cuda")
        return x.normal_(0.0, scale, generator=gen) if not torch.is_tensor(scale) else x.normal_(0.0, 1.0, generator=gen).mul_(scale)

    lo, hi = math.log(1e-4), math.log(1e-1)
    if kind == "segments":
        off = _segments(c)
        rng = random.Random(seed + 5)
        s = torch.empty(P, device="cuda")
        for i in range(c["S"]):
            s[off[i]:off[i + 1]] = math.exp(rng.uniform(lo, hi))
    else:
        s = torch.empty(P, device="cuda").uniform_(lo, hi, generator=gen).exp_()
    x = {"theta": normal(0.05)}
    if c.get("rule") != "sasgd":
        # averages of a running server: b scatters around 0 by s sqrt((1 - gamma) / (1 + gamma)),
        # n by about as much around s^2, and v follows them
        x["b"] = normal(s).mul_(math.sqrt((1 - GAMMA) / (1 + GAMMA)))
        x["n"] = normal(0.15).add_(1.0).clamp_(0.3, 1.7).mul_(s).mul_(s).addcmul_(x["b"], x["b"])
        x["v"] = (x["n"] - x["b"] * x["b"]).clamp_(min=0).add_(EPS).rsqrt_()
    m = normal(1e-3)
    count = {"dense": c.get("K"), "step": c.get("K", 0) + 1, "pushes": c.get("B"), "fetch": 0}.get(kind, 1)
    x["grads"] = [normal(s).add_(m) for _ in range(count)]
    if "f" in c:
        # the threshold that sends a fraction f of the parameters (for "segments": of the tensors) on average
        v = x["v"][: 1 << 16].double().cpu() if kind != "segments" else x["v"].mean().double().cpu().reshape(1)
        a, b = 1e-6, 1e9
        for _ in range(60):
            mid = math.sqrt(a * b)
            a, b = (mid, b) if float((v / (v + mid)).mean()) > c["f"] else (a, mid)
        x["c"] = float(np.float32(a))
    if kind == "step":
        # the push that the previous step selected
        idx = torch.nonzero(torch.empty(P, device="cuda").uniform_(0.0, 1.0, generator=gen) < c["f"]).reshape(-1)
        x["push_idx"] = idx.int()
        x["push_val"] = normal(s)[idx]
    if kind == "cached":
        x["cache"] = normal(s)
    if kind == "fetch":
        x["copy"] = normal(0.05)
    return x


def prepare(case, seed):
    c, P = case, case["P"]
    x = _inputs(c, seed)
    st = dict(c, x=x, seed=seed)
    i32 = dict(device="cuda", dtype=torch.int32)
    last_T = torch.empty(P, **i32)
    stats = [x.get(k) for k in ("n", "b", "v")]
    keep = [t.clone() if t is not None else None for t in stats]   # fasgd_init_state fills the arrays
    server = fa.fasgd_init_state(x["theta"], *keep, last_T, lam=c["lam"], alpha=_alpha(c), gamma=GAMMA, beta=BETA,
                                 eps=EPS, math_mode=fa.MATH_IEEE if c.get("math") == "ieee" else fa.MATH_FAST)
    for dst, src in zip(keep, stats):
        if dst is not None:
            dst.copy_(src)
    for k in ("n", "b", "v"):
        x.pop(k, None)
    server.c.T, server.c.dense_T = T0, T0 - 1
    st["server"] = server
    st["clients"], st["delays"] = _arrivals(c, seed, max(c.get("K", 1), c.get("B", 1)) + 1)
    B = c.get("B", 1)
    if c["kind"] not in ("dense", "segments"):
        shape = (B, P) if c["kind"] == "pushes" else (P,)
        st["idx"] = torch.zeros(shape, **i32)
        st["val"] = torch.zeros(shape, device="cuda")
        st["cnt"] = torch.zeros(B, device="cuda", dtype=torch.int64)
        L = fa.bfasgd_list_index_length(P)
        st["seg"] = torch.zeros((B, L) if c["kind"] == "pushes" else (L,), **i32)
        st["ws"] = torch.empty(B * fa.bfasgd_workspace_bytes(P), device="cuda", dtype=torch.uint8)
    if c["kind"] == "step":
        m = x["push_idx"].numel()
        st["idx"][:m] = x["push_idx"]
        st["val"][:m] = x["push_val"]
        st["cnt"].fill_(m)
        edges = torch.arange(L, device="cuda") * 256
        st["seg"].copy_(torch.searchsorted(x["push_idx"], edges.clamp_(max=P).int(), right=False))
        del x["push_idx"], x["push_val"]
    if c["kind"] == "segments":
        st["off"] = _segments(c)
        st["send"] = torch.zeros(c["S"], device="cuda", dtype=torch.uint8)
        st["ws"] = torch.empty(fa.bfasgd_segments_workspace_bytes(P, c["S"]), device="cuda", dtype=torch.uint8)
    return st


def _server_arrays(server):
    return {k: server.tensors[k] for k in ("theta", "n", "b", "v", "last_T") if server.tensors[k] is not None}


def run(st):
    kind, sv, x, T = st["kind"], st["server"], st["x"], st["server"].T
    clients, delays = st["clients"], st["delays"]
    if kind == "dense":
        K = st["K"]
        apply = fa.sasgd_apply_updates if st["rule"] == "sasgd" else fa.fasgd_apply_updates
        apply(sv, x["grads"], clients[:K], [T + k - delays[k] for k in range(K)])
        return _server_arrays(sv)
    if kind == "step":
        K = st["K"]
        fa.fasgd_apply_with_push_and_select(
            sv, st["idx"], st["val"], st["cnt"], st["seg"], clients[K], T - delays[K], x["grads"][:K], clients[:K],
            [T + 1 + k - delays[k] for k in range(K)], x["grads"][K], clients[K], x["c"], EPS_C, st["seed"],
            st["idx"], st["val"], st["cnt"], st["seg"], st["ws"])
        return dict(_server_arrays(sv), idx=st["idx"], val=st["val"], cnt=st["cnt"], seg=st["seg"])
    if kind == "pushes":
        B = st["B"]
        fa.bfasgd_select_compact_batch(sv, x["grads"], x["c"], EPS_C, st["seed"], [T + b for b in range(B)],
                                       clients[:B], st["idx"], st["val"], st["cnt"], st["ws"], seg_start=st["seg"])
        fa.fasgd_apply_pushes(sv, st["idx"], st["val"], st["cnt"], st["seg"], clients[:B],
                              [T + b - delays[b] for b in range(B)])
        return dict(_server_arrays(sv), idx=st["idx"], val=st["val"], cnt=st["cnt"], seg=st["seg"])
    if kind == "segments":
        fa.bfasgd_decide_segments(sv, st["off"], x["c"], EPS_C, st["seed"], T, clients[0], st["send"], st["ws"])
        fa.bfasgd_apply_segments(sv, x["grads"][0], st["off"], st["send"], clients[0], T - delays[0])
        return dict(_server_arrays(sv), send=st["send"])
    # the index is asked for where the consumer uses it
    indexed = kind in ("select", "cached") or (kind == "fetch" and 4 * st["P"] > 256e6)
    seg = st["seg"] if indexed else None
    values = sv.tensors["theta"] if kind == "fetch" else x["grads"][0]
    fa.bfasgd_select_compact(sv, values, x["c"], EPS_C, st["seed"], T, clients[0], st["idx"], st["val"], st["cnt"],
                             st["ws"], seg_start=seg)
    out = {"idx": st["idx"], "val": st["val"], "cnt": st["cnt"]}
    if indexed:
        out["seg"] = seg
    if kind == "select":
        return out
    if kind == "fetch":
        fa.bfasgd_apply_fetch(x["copy"], st["idx"], st["val"], st["cnt"], seg_start=seg)
        return dict(out, copy=x["copy"])
    if kind == "cached":
        fa.bfasgd_apply_cached(sv, st["idx"], st["val"], st["cnt"], x["cache"], clients[0], T - delays[0], seg_start=seg)
        return dict(_server_arrays(sv), cache=x["cache"], **out)
    fa.bfasgd_apply_sparse(sv, st["idx"], st["val"], st["cnt"], clients[0], T - delays[0])
    return dict(_server_arrays(sv), **out)


def work(case):
    """Bytes: each input read once and each output written once (the state is both).  About 14 operations an update."""
    c, P, kind = case, case["P"], case["kind"]
    f = c.get("f", 0.0)
    m = f * P
    if kind == "dense":
        state = 8 if c["rule"] == "sasgd" else 32
        return {"bytes": P * (state + 4 * c["K"]), "flops": (2 if c["rule"] == "sasgd" else 14) * P * c["K"]}
    if kind == "step":
        return {"bytes": P * (32 + 4 * (c["K"] + 1)) + 16 * m + 8 * (P / 256), "flops": 14 * (P * c["K"] + m) + 10 * P}
    if kind == "pushes":
        listed_once = (1 - (1 - f) ** c["B"]) * P
        return {"bytes": 4 * P + c["B"] * (4 * P + 8 * m + 4 * (P / 256)) + 36 * listed_once,
                "flops": c["B"] * (14 * m + 10 * P)}
    if kind == "segments":
        return {"bytes": 4 * P + f * 40 * P, "flops": P + 14 * f * P}
    select = 8 * P + 8 * m
    if kind == "select":
        return {"bytes": select + 4 * (P / 256), "flops": 10 * P}
    if kind == "fetch":
        return {"bytes": select + 4 * m, "flops": 10 * P}
    if kind == "cached":
        return {"bytes": select + 36 * P - 4 * P + 4 * m, "flops": 24 * P}
    return {"bytes": select + 36 * m, "flops": 10 * P + 14 * m}


def tolerance(case):
    """Selections and list copies are decided and copied bit for bit; the state is fp32 (fast math: reciprocals of
    about 1 ulp), at most 32 updates deep: up to 1.9e-7 from the 64-bit reference."""
    if case["kind"] in ("select", "fetch"):
        return "exact"
    return {"rel": 1e-6}


# ---------------------------------------------------------------- 64-bit reference

M32 = 0xFFFFFFFF


def _philox(x0, x1, x2, x3, k0, k1):
    """Philox4x32-10 on int64 tensors or ints holding 32-bit words."""
    for i in range(10):
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57
        h0, h1 = (p0 >> 32) & M32, (p1 >> 32) & M32
        x0, x1, x2, x3 = h1 ^ x1 ^ k0, p1 & M32, h0 ^ x3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return x0, x1, x2, x3


def _sent(v, c, seed, T, client, lo, hi):
    """The transmit decisions of parameters [lo, hi) (lo a multiple of 4), from their fp32 v."""
    q = torch.arange(lo // 4, (hi + 3) // 4, device=v.device, dtype=torch.int64)
    w = _philox(q, torch.zeros_like(q), torch.full_like(q, T), torch.full_like(q, client), seed & M32, seed >> 32)
    r = (torch.stack(w, 1).reshape(-1)[: hi - lo] >> 8).double() * 2.0 ** -24
    t = v[lo:hi] + torch.tensor(EPS_C, device=v.device, dtype=torch.float32)
    u = t + torch.tensor(c, device=v.device, dtype=torch.float32)
    return r * u.double() < t.double()


def _update(s, g, c, tau, where=None):
    """One server update of the 64-bit state slices s in place, restricted to `where`."""
    gamma, beta, eps, alpha = (float(np.float32(z)) for z in (GAMMA, BETA, EPS, _alpha(c)))
    rate = alpha / max(tau, 1)
    g = g.double()
    if c.get("rule") == "sasgd":
        s["theta"] -= rate * g
        return
    n = gamma * s["n"] + (1 - gamma) * g * g
    b = gamma * s["b"] + (1 - gamma) * g
    v = beta * s["v"] + (1 - beta) / torch.sqrt((n - b * b).clamp_(min=0) + eps)
    new = {"n": n, "b": b, "v": v, "theta": s["theta"] - rate / v * g}
    for k, y in new.items():
        s[k] = y if where is None else torch.where(where, y, s[k])


def exact(case, seed):
    c, P, kind = case, case["P"], case["kind"]
    if kind in ("select", "fetch"):
        return None     # whole numbers and bit copies
    x = _inputs(c, seed)
    clients, delays = _arrivals(c, seed, max(c.get("K", 1), c.get("B", 1)) + 1)
    names = ("theta",) if c.get("rule") == "sasgd" else ("theta", "n", "b", "v")
    out = {k: torch.empty(P, device="cuda", dtype=torch.float64) for k in names}
    if kind == "cached":
        out["cache"] = torch.empty(P, device="cuda", dtype=torch.float64)
    off, sends = None, None
    if kind == "segments":
        off = _segments(c)
        sends = []
        for i in range(c["S"]):
            mean = float(x["v"][off[i]:off[i + 1]].double().mean())
            w = _philox(i, 0x80000000, T0, clients[0], seed & M32, seed >> 32)
            t = mean + float(np.float32(EPS_C))
            sends.append((w[0] >> 8) * 2.0 ** -24 * (t + x["c"]) < t)
    if kind == "step":
        pushed = torch.zeros(P, device="cuda", dtype=torch.bool)
        pushed[x["push_idx"].long()] = True
        values = torch.zeros(P, device="cuda")
        values[x["push_idx"].long()] = x["push_val"]
    span = 1 << 25
    for lo in range(0, P, span):
        hi = min(P, lo + span)
        s = {k: x[k][lo:hi].double() for k in names}
        g = [t[lo:hi] for t in x["grads"]]
        if kind == "dense":
            for k in range(c["K"]):
                _update(s, g[k], c, delays[k])
        elif kind == "step":
            _update(s, values[lo:hi], c, delays[c["K"]], pushed[lo:hi])
            for k in range(c["K"]):
                _update(s, g[k], c, delays[k])
        elif kind == "pushes":
            for b in range(c["B"]):
                _update(s, g[b], c, delays[b], _sent(x["v"], x["c"], seed, T0 + b, clients[b], lo, hi))
        elif kind == "push":
            _update(s, g[0], c, delays[0], _sent(x["v"], x["c"], seed, T0, clients[0], lo, hi))
        elif kind == "cached":
            cache = torch.where(_sent(x["v"], x["c"], seed, T0, clients[0], lo, hi), g[0], x["cache"][lo:hi])
            _update(s, cache, c, delays[0])
            out["cache"][lo:hi] = cache
        elif kind == "segments":
            where = torch.zeros(hi - lo, device="cuda", dtype=torch.bool)
            for i in range(c["S"]):
                if sends[i]:
                    where[max(0, off[i] - lo):max(0, off[i + 1] - lo)] = True
            _update(s, g[0], c, delays[0], where)
        for k in names:
            out[k][lo:hi] = s[k]
    if c.get("rule") == "sasgd":
        return {"theta": out["theta"], "last_T": None}
    lists = {} if kind in ("dense", "segments") else {"idx": None, "val": None, "cnt": None}
    if kind in ("step", "pushes", "cached"):
        lists["seg"] = None
    if kind == "segments":
        lists["send"] = None
    return dict(out, last_T=None, **lists)
