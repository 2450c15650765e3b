"""The work that a user has this library do, as cases that can be measured.

One case is one MoE layer of a training program on one GPU: `prepare` makes what the program
holds before the call (context, buffers, weights in the replica slots, optimizer state, a batch),
`run` is one pass through the public entry points in the order of a training iteration.

kinds   step       route, dispatch, expert forward, combine, their backwards, next placement,
                   optimizer step written into the next placement's slots
        forward    route, dispatch (dropless, or under a capacity factor), expert forward, combine
        backward   combine backward, expert backward, dispatch backward, route backward
        slots      expert backward with one weight gradient per replica slot, then the replica
                   all-reduce (the gradient exchange between a class's replicas)
        optimizer  next placement and the optimizer step alone
        router     the gate network: scores of every token, and its backward behind the dispatch's

Sizes are those of workloads/configs.py (c1 .. c5) and of the tests' ragged shapes.
"""
import math

import numpy as np
import torch

import paper_2504_19925_amd as symi

KINDS = ("step", "forward", "backward", "slots", "optimizer", "router")


def _case(kind, dtype, E, k, d, f, T, S, N, **kw):
    c = {"kind": kind, "dtype": dtype, "E": E, "k": k, "d": d, "f": f, "T": T, "S": S, "N": N,
         "zipf": 0.0,       # class scores -2 s log(rank), ranking shuffled by the seed
         "hot": 0.0,        # extra score of one class
         "drift": 0.0,      # class scores N(0, drift^2)
         "noise": 1.0,      # per-token noise of the scores
         "renorm": 1,       # gates of a token sum to 1
         "active": False,   # the *_active pair: classes without tokens are not written or read
         "capacity": 0.0}   # capacity factor of the dispatch, 0 = dropless
    c.update(kw)
    return c


def listed():
    named = [
        # the smallest iteration anybody runs: a single-precision layer for debugging and reference
        # runs (configuration c1); its launches are short, so latency and their number count
        ("c1 step f32", _case("step", "f32", 8, 2, 128, 256, 1024, 16, 4, zipf=1.2, noise=0.23)),
        # the same precision at sizes that are no multiple of any tile, three choices per token
        ("ragged step f32", _case("step", "f32", 24, 3, 328, 872, 2999, 36, 4, zipf=0.5)),
        # a handful of tokens through a narrow layer: nothing but launches and host work
        ("tiny forward", _case("forward", "bf16", 16, 2, 128, 256, 64, 24, 8, zipf=1.2)),
        # validation on a short batch with c2's widths: a few rows per expert, weights dominate
        ("short forward", _case("forward", "bf16", 64, 2, 1024, 4096, 200, 96, 8, zipf=0.5)),
        # c2: strong skew, most classes without tokens, a quarter of the step is the optimizer
        ("c2 step", _case("step", "bf16", 64, 2, 1024, 4096, 8192, 96, 8, zipf=1.2, active=True)),
        # widths and batch that are no multiple of a tile, gates not renormalised
        ("ragged backward", _case("backward", "bf16", 12, 3, 1160, 2744, 5003, 20, 4, zipf=0.5, renorm=0)),
        # c3: few wide experts, one of them with about 40 % of the assignments
        ("c3 step", _case("step", "bf16", 8, 2, 4096, 14336, 16384, 16, 8, hot=3.0, noise=1.7)),
        # c4: many narrow experts, six choices, popularity that drifted for some ten iterations
        ("c4 step", _case("step", "bf16", 64, 6, 2048, 1408, 32768, 128, 16, drift=0.95)),
        # c4's forward when a slot may take no more than its share
        ("c4 capacity forward", _case("forward", "bf16", 64, 6, 2048, 1408, 32768, 128, 16, drift=0.95,
                                      capacity=1.0)),
        # c4's widths on a smaller batch with the gradient exchange drawn out slot by slot
        ("slot gradients", _case("slots", "bf16", 64, 6, 2048, 1408, 8192, 128, 16, drift=0.95)),
        # c5: the largest batch and layer, near-uniform popularity
        ("c5 step", _case("step", "bf16", 128, 8, 4096, 2048, 65536, 256, 32, zipf=0.5, active=True)),
        # c5's gate network
        ("c5 router", _case("router", "bf16", 128, 8, 4096, 2048, 65536, 256, 32, zipf=0.5)),
    ]
    return [dict(c, name=name) for name, c in named]


def _flops(c):
    A = c["T"] * c["k"]
    each = 2.0 * A * c["d"] * c["f"]
    return {"step": 9, "forward": 3, "backward": 6, "slots": 6, "optimizer": 0}.get(c["kind"], 0) * each


def _state_bytes(c):
    w = 2 if c["dtype"] == "bf16" else 4
    A, d, f = c["T"] * c["k"], c["d"], c["f"]
    if c["kind"] == "router":
        return A * d * w + 3 * c["T"] * d * w + 8 * c["E"] * c["T"]
    weights = c["S"] * 3 * d * f * w
    grads = (c["S"] if c["kind"] == "slots" else c["E"]) * 3 * d * f * 4
    acts = A * (4 * d + 5 * f) * w
    return weights + grads + (0 if c["kind"] == "optimizer" else acts)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    while True:
        kind = rng.choice(("step", "step", "step", "forward", "forward", "backward", "slots", "optimizer", "router"))
        dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        if dtype == "f32":      # single precision: reference and debugging sizes
            E, k = rng.choice((4, 8, 16, 24)), rng.randint(1, 4)
            d, f = 8 * round(_log(rng, 8, 64)), 8 * round(_log(rng, 16, 160))
            T = round(_log(rng, 64, 8192))
        else:
            E, k = rng.choice((8, 12, 16, 48, 64, 128)), rng.randint(1, 8)
            d, f = 8 * round(_log(rng, 16, 512)), 8 * round(_log(rng, 32, 1792))
            T = round(_log(rng, 16, 65536))
        N = rng.choice((1, 2, 4, 8, 16, 32))
        while (3 * d * f) % (8 * N):
            N //= 2
        S = N * math.ceil(E * rng.uniform(1.0, 2.5) / N)
        c = _case(kind, dtype, E, k, d, f, T, S, N, renorm=rng.randint(0, 1), active=rng.random() < 0.5)
        skew = rng.choice(("zipf", "zipf", "hot", "drift"))
        c[skew] = round({"zipf": rng.uniform(0.0, 1.2), "hot": rng.uniform(1.0, 3.0), "drift": rng.uniform(0.1, 1.3)}[skew], 3)
        if kind == "forward" and rng.random() < 0.4:
            c["capacity"] = round(rng.uniform(0.8, 1.5), 3)
        if _flops(c) > (3e11 if dtype == "f32" else 3.5e13) or _state_bytes(c) > 30e9:
            continue
        return c


class _State:
    """What the program keeps between iterations, and the batch of this one."""


def _bias(c, g):
    E = c["E"]
    if c["zipf"]:
        rank = torch.arange(1, E + 1, dtype=torch.float64)
        return ((-2.0 * c["zipf"]) * torch.log(rank))[torch.randperm(E, generator=g)].float()
    if c["drift"]:
        return (torch.randn(E, generator=g, dtype=torch.float64) * c["drift"]).float()
    b = torch.zeros(E)
    b[int(torch.randint(E, (1,), generator=g))] = c["hot"]
    return b


def prepare(case, seed):
    c = dict(case)
    s = _State()
    s.case = c
    dev = torch.device("cuda")
    gh = torch.Generator().manual_seed(seed * 7919 + 1)
    gd = torch.Generator(device=dev).manual_seed(seed * 7919 + 2)
    E, k, d, f, T, S, N = (c[n] for n in ("E", "k", "d", "f", "T", "S", "N"))
    A = T * k
    s.cfg = symi.SymiCfg.make(T, E, k, d, f, S, N, seed % N, c["dtype"], c["renorm"])
    s.ctx = symi.symi_create(s.cfg)
    dt = s.cfg.torch_dtype
    s.ws = torch.empty(symi.symi_workspace_bytes(s.cfg), dtype=torch.uint8, device=dev)

    def new(*n, dtype=dt):
        return torch.zeros(*n, dtype=dtype, device=dev)

    def normal(*n, std=1.0, dtype=dt):
        return torch.randn(*n, generator=gd, dtype=dtype, device=dev).mul_(std)

    i32, f32 = torch.int32, torch.float32
    bias = _bias(c, gh).to(dev)
    if c["kind"] == "router":
        s.X, s.dXp, s.dX = normal(T, d), normal(A, d), new(T, d)
        s.roa = torch.randperm(A, generator=gd, device=dev).to(i32)
        s.Wr, s.b = normal(E, d, std=0.02), bias
        s.logits, s.dlogits = new(T, E, dtype=f32), normal(T, E, std=0.01, dtype=f32)
        s.dWr, s.db = new(E, d, dtype=f32), new(E, dtype=f32)
        return s

    # popularity of the batch before decides where the replicas are now
    def scores():
        return normal(T, E, std=c["noise"], dtype=f32).add_(bias)

    s.counts, s.placement, s.first = new(E, dtype=i32), new(S, dtype=i32), new(E + 1, dtype=i32)
    s.counts2, s.placement2, s.first2 = new(E, dtype=i32), new(S, dtype=i32), new(E + 1, dtype=i32)
    s.idx, s.gate, s.hist = new(T, k, dtype=i32), new(T, k, dtype=f32), new(E, dtype=i32)
    symi.symi_route(s.ctx, scores(), s.idx, s.gate, s.hist)
    symi.symi_place(s.ctx, s.hist, s.counts, s.placement, s.first)

    if c["kind"] in ("step", "optimizer"):
        per = 3 * d * f // N
        lo, n1 = per * (seed % N), 2 * f * d
    W1c, W2c = normal(E, 2 * f, d, std=0.02), normal(E, d, f, std=0.02)
    at = s.placement.long()
    s.W1, s.W2 = W1c.index_select(0, at), W2c.index_select(0, at)
    if c["kind"] in ("step", "optimizer"):
        part = []
        if lo < n1:
            part.append(W1c.view(E, -1)[:, lo:min(lo + per, n1)])
        if lo + per > n1:
            part.append(W2c.view(E, -1)[:, max(lo - n1, 0):lo + per - n1])
        s.master = torch.cat(part, 1).float().contiguous()
        # moments of a run that has been going on for a while
        s.m = normal(E, per, std=0.3, dtype=f32)
        s.v = normal(E, per, dtype=f32).square_().add_(0.1)
        s.step = 1000
    del W1c, W2c
    if c["kind"] == "optimizer":
        symi.symi_route(s.ctx, scores(), s.idx, s.gate, s.hist)
        s.dW1, s.dW2 = normal(E, 2 * f, d, dtype=f32), normal(E, d, f, dtype=f32)
        return s

    s.X, s.logits = normal(T, d), scores()
    s.roa, s.aor, s.offs = new(A, dtype=i32), new(A, dtype=i32), new(S + 1, dtype=i32)
    s.Xp, s.UV, s.H, s.Yp, s.Y = new(A, d), new(A, 2 * f), new(A, f), new(A, d), new(T, d)
    s.cap = symi.symi_slot_capacity(s.cfg, c["capacity"]) if c["capacity"] else 0
    if c["kind"] != "forward":
        s.dY, s.dYp, s.dXp, s.dX = normal(T, d), new(A, d), new(A, d), new(T, d)
        s.dgate, s.dlogits = new(T, k, dtype=f32), new(T, E, dtype=f32)
        G = S if c["kind"] == "slots" else E
        s.dW1, s.dW2 = new(G, 2 * f, d, dtype=f32), new(G, d, f, dtype=f32)
    if c["kind"] in ("backward", "slots"):
        _forward(s)
    if c["kind"] == "slots":
        symi.symi_combine_bwd(s.ctx, s.dY, s.Yp, s.roa, s.gate, s.dYp, s.dgate)
    return s


def _forward(s):
    symi.symi_route(s.ctx, s.logits, s.idx, s.gate, s.hist)
    if s.cap:
        symi.symi_dispatch_capacity(s.ctx, s.cap, s.X, s.idx, s.hist, s.counts, s.first, s.roa, s.aor, s.offs, s.Xp, s.ws)
    else:
        symi.symi_dispatch(s.ctx, s.X, s.idx, s.hist, s.counts, s.first, s.roa, s.aor, s.offs, s.Xp, s.ws)
    symi.symi_expert_fwd(s.ctx, s.Xp, s.offs, s.W1, s.W2, s.UV, s.H, s.Yp, s.ws)
    symi.symi_combine(s.ctx, s.Yp, s.roa, s.gate, s.Y)
    return {"idx": s.idx, "gate": s.gate, "hist": s.hist, "rows": s.roa, "offsets": s.offs, "Y": s.Y,
            "Xp": s.Xp, "UV": s.UV, "H": s.H, "Yp": s.Yp}


def _backward(s):
    symi.symi_combine_bwd(s.ctx, s.dY, s.Yp, s.roa, s.gate, s.dYp, s.dgate)
    bwd = symi.symi_expert_bwd_active if s.case["active"] else symi.symi_expert_bwd
    bwd(s.ctx, s.dYp, s.Xp, s.UV, s.H, s.offs, s.first, s.W1, s.W2, s.dXp, s.dW1, s.dW2, s.ws)
    symi.symi_dispatch_bwd(s.ctx, s.dXp, s.roa, s.dX)
    symi.symi_route_bwd(s.ctx, s.logits, s.idx, s.gate, s.dgate, s.dlogits)
    return {"dX": s.dX, "dlogits": s.dlogits, "dW1": s.dW1, "dW2": s.dW2}


def _optimizer(s):
    hp = symi.SymiAdam(1e-4, 0.9, 0.999, 1e-8, 0.01, 1.0, s.step)
    s.step += 1
    symi.symi_place(s.ctx, s.hist, s.counts2, s.placement2, s.first2)
    if s.case["active"] and s.case["kind"] == "step":
        symi.symi_adam_to_replicas_active(s.ctx, hp, s.dW1, s.dW2, s.master, s.m, s.v, s.offs, s.first, s.first2, s.W1, s.W2)
    else:
        symi.symi_adam_to_replicas(s.ctx, hp, s.dW1, s.dW2, s.master, s.m, s.v, s.first2, s.W1, s.W2)
    out = {"placement": s.placement2, "master": s.master, "m": s.m, "v": s.v, "W1": s.W1, "W2": s.W2}
    # the next iteration dispatches with the placement just written
    s.counts, s.counts2 = s.counts2, s.counts
    s.placement, s.placement2 = s.placement2, s.placement
    s.first, s.first2 = s.first2, s.first
    return out


def run(s):
    kind = s.case["kind"]
    if kind == "forward":
        return _forward(s)
    if kind == "backward":
        return _backward(s)
    if kind == "optimizer":
        return _optimizer(s)
    if kind == "slots":
        symi.symi_expert_bwd_slots(s.ctx, s.dYp, s.Xp, s.UV, s.H, s.offs, s.first, s.W1, s.W2, s.dXp, s.dW1, s.dW2, s.ws)
        symi.symi_replica_allreduce(s.ctx, s.first, 1.0, s.dW1, s.dW2)
        return {"dXp": s.dXp, "dW1": s.dW1, "dW2": s.dW2}
    if kind == "router":
        symi.symi_router_fwd(s.ctx, s.X, s.Wr, s.b, s.logits)
        symi.symi_dispatch_bwd(s.ctx, s.dXp, s.roa, s.dX)
        symi.symi_router_bwd(s.ctx, s.X, s.Wr, s.dlogits, s.dWr, s.db, s.dX, s.ws)
        return {"logits": s.logits, "dWr": s.dWr, "db": s.db, "dX": s.dX}
    out = {**_forward(s), **_backward(s), **_optimizer(s)}
    for n in ("Xp", "UV", "H", "Yp"):       # scratch of the program once the backward is through
        del out[n]
    return out


def _occupied(c):
    """Classes and slots that get rows, about: from the popularity of a sample of tokens."""
    E, k, T, S = c["E"], c["k"], c["T"], c["S"]
    r = np.random.RandomState(0)
    b = _bias(c, torch.Generator().manual_seed(0)).numpy()
    n = min(T, 4096)
    z = r.randn(n, E) * c["noise"] + b
    h = np.bincount(np.argpartition(-z, k - 1, 1)[:, :k].ravel(), minlength=E) * (T / n)
    classes = int((h > 0).sum())
    reps = np.maximum(1, np.floor(h / h.sum() * (S - (E - classes))))   # a class without tokens keeps one slot
    return classes, int(min(np.minimum(reps, np.ceil(h)).sum(), S - (E - classes)))


def work(case):
    """Inputs of the pass read once, its results written once; buffers that only carry values from
    one stage to the next are not counted."""
    c = dict(case)
    E, k, d, f, T, S, N = (c[n] for n in ("E", "k", "d", "f", "T", "S", "N"))
    w = 2 if c["dtype"] == "bf16" else 4
    A, P = T * k, 3 * d * f
    if c["kind"] == "router":
        return {"bytes": A * d * w + 2 * T * d * w + E * d * (w + 4) + 2 * T * E * 4 + A * 4, "flops": 6.0 * T * d * E}
    cls, slots = (E, S) if c["kind"] == "optimizer" else _occupied(c)
    ints = 3 * A * 4 + (E + S) * 4
    fwd = 2 * T * d * w + T * E * 4 + slots * P * w + ints
    # the saved u, v, h and the permuted tokens, expert outputs and their gradients are the
    # backward's inputs; inside a step they are not
    saved = A * (2 * d + 3 * f) * w
    grads = (cls if c["active"] else E) * P * 4
    bwd = 2 * T * d * w + 2 * T * E * 4 + slots * P * w + grads + A * 12
    opt = E * (P // N) * 24 + (cls if c["active"] else E) * (P // N) * 4 + S * (P // N) * w
    total = {"step": fwd + bwd + opt, "forward": fwd, "backward": bwd + saved, "optimizer": opt,
             "slots": A * (3 * d + 3 * f) * w + slots * P * w + S * P * 4}[c["kind"]]
    return {"bytes": float(total), "flops": _flops(c)}


def tolerance(case):
    """Distances from the same path in binary64 (relative 2-norm / largest over the rms), measured on
    the listed and on drawn shapes: single precision 2.8e-7 / 5e-6; bf16 3.9e-3 / 0.14 (largest in
    the weight gradients of classes with few rows); the optimizer's bf16 slots differ where the
    fresh weight sits at a rounding boundary."""
    if case["dtype"] == "f32":
        return {"rel": 1.5e-6, "max": 3e-5}
    if case["kind"] == "optimizer":
        return {"rel": 1e-4, "max": 1e-2}
    return {"rel": 1e-2, "max": 0.4}


# ---- the same results in binary64, in plain torch, from the inputs that `prepare` makes

def _exact_place(hist, S):
    """Slots of the classes by popularity: floors, then shrink the most / grow the least rounded up."""
    pop = [max(int(h), 0) for h in hist]
    P = sum(pop)
    if P == 0:
        pop, P = [1] * len(pop), len(pop)
    n = [max(1, p * S // P) for p in pop]
    diff = [c * P - p * S for c, p in zip(n, pop)]
    while sum(n) > S:
        i = max((i for i in range(len(n)) if n[i] > 1), key=lambda i: (diff[i], -i))
        n[i] -= 1
        diff[i] -= P
    while sum(n) < S:
        i = min(range(len(n)), key=lambda i: (diff[i], i))
        n[i] += 1
        diff[i] += P
    return n


def _exact_forward(s):
    c, D, dev = s.case, torch.float64, s.X.device
    E, k, T, A = c["E"], c["k"], c["T"], c["T"] * c["k"]
    s.p = torch.softmax(s.logits.to(D), 1)
    idx = torch.sort(s.logits, dim=1, descending=True, stable=True).indices[:, :k].contiguous()
    gate = s.p.gather(1, idx)
    if c["renorm"]:
        gate = gate / gate.sum(1, keepdim=True)
    cls = idx.reshape(-1)
    order = torch.argsort(cls, stable=True)      # rows: assignments by class, in their own order
    hist = torch.bincount(cls, minlength=E)
    kept = hist
    if s.cap:
        begin = hist.cumsum(0) - hist
        quota = s.cap * s.counts.to(torch.int64)
        rank = torch.arange(A, device=dev) - begin[cls[order]]
        order = order[rank < quota[cls[order]]]
        kept = torch.minimum(hist, quota)
    R = order.numel()
    roa = torch.full((A,), -1, dtype=torch.int64, device=dev)
    roa[order] = torch.arange(R, device=dev)
    s.xidx, s.xgate, s.xroa, s.xhist, s.rows = idx, gate, roa.view(T, k), hist.tolist(), kept.tolist()
    f = c["f"]
    Xp, UV, H, Yp = (torch.zeros(A, n, dtype=D, device=dev) for n in (c["d"], 2 * f, f, c["d"]))
    Xp[:R] = s.X.to(D)[order // k]
    for e, o, n in _classes(s):
        W1, W2 = _weights(s, e)
        UV[o:o + n] = Xp[o:o + n] @ W1.t()
        u, v = UV[o:o + n, :f], UV[o:o + n, f:]
        H[o:o + n] = u * torch.sigmoid(u) * v
        Yp[o:o + n] = H[o:o + n] @ W2.t()
    g = torch.where(s.xroa >= 0, gate, torch.zeros_like(gate))
    Y = torch.zeros(T, c["d"], dtype=D, device=dev)
    for j in range(k):
        Y += g[:, j:j + 1] * Yp[s.xroa[:, j].clamp(min=0)]
    s.xXp, s.xUV, s.xH, s.xYp = Xp, UV, H, Yp
    return {"idx": None, "gate": gate, "hist": None, "rows": None, "offsets": None, "Y": Y,
            "Xp": Xp, "UV": UV, "H": H, "Yp": Yp}


def _classes(s):
    o = 0
    for e, n in enumerate(s.rows):
        if n:
            yield e, o, n
        o += n


def _weights(s, e):
    q = int(s.first[e])
    return s.W1[q].double(), s.W2[q].double()


def _exact_experts(s, dYp):
    c, D = s.case, torch.float64
    E, d, f = c["E"], c["d"], c["f"]
    dXp = torch.zeros_like(dYp)
    dW1, dW2 = torch.zeros(E, 2 * f, d, dtype=D, device=dYp.device), torch.zeros(E, d, f, dtype=D, device=dYp.device)
    for e, o, n in _classes(s):
        W1, W2 = _weights(s, e)
        dy, u, v = dYp[o:o + n], s.xUV[o:o + n, :f], s.xUV[o:o + n, f:]
        dh, sg = dy @ W2, torch.sigmoid(u)
        duv = torch.cat((dh * v * sg * (1 + u * (1 - sg)), dh * u * sg), 1)
        dXp[o:o + n] = duv @ W1
        dW1[e], dW2[e] = duv.t() @ s.xXp[o:o + n], dy.t() @ s.xH[o:o + n]
    return dXp, dW1, dW2


def _exact_backward(s):
    c, D = s.case, torch.float64
    dY = s.dY.to(D)
    dYp, dgate = torch.zeros_like(s.xYp), torch.zeros_like(s.xgate)
    for j in range(c["k"]):
        at = s.xroa[:, j]
        dYp[at] = s.xgate[:, j:j + 1] * dY
        dgate[:, j] = (dY * s.xYp[at]).sum(1)
    dXp, dW1, dW2 = _exact_experts(s, dYp)
    dX = torch.zeros_like(dY)
    for j in range(c["k"]):
        dX += dXp[s.xroa[:, j]]
    ps = s.p.gather(1, s.xidx)
    if c["renorm"]:
        dgate = (dgate - (dgate * s.xgate).sum(1, keepdim=True)) / ps.sum(1, keepdim=True)
    dp = torch.zeros_like(s.p).scatter_(1, s.xidx, dgate)
    return {"dX": dX, "dlogits": s.p * (dp - (dgate * ps).sum(1, keepdim=True)), "dW1": dW1, "dW2": dW2}


def _exact_optimizer(s, hist, dW1, dW2):
    c, D = s.case, torch.float64
    E, n1 = c["E"], 2 * c["f"] * c["d"]
    per = 3 * c["d"] * c["f"] // c["N"]
    lo = per * s.cfg.shard
    g = torch.cat((dW1.reshape(E, -1)[:, min(lo, n1):min(lo + per, n1)],
                   dW2.reshape(E, -1)[:, max(lo - n1, 0):max(lo + per - n1, 0)]), 1).to(D)
    b1, b2, lr, eps, wd = (float(np.float32(x)) for x in (0.9, 0.999, 1e-4, 1e-8, 0.01))
    m, v = b1 * s.m.to(D) + (1 - b1) * g, b2 * s.v.to(D) + (1 - b2) * g * g
    w = s.master.to(D)
    w = w - lr * (m / (1 - b1 ** s.step) / (torch.sqrt(v / (1 - b2 ** s.step)) + eps) + wd * w)
    at = torch.repeat_interleave(torch.arange(E), torch.tensor(_exact_place(hist, c["S"]))).to(w.device)
    W1, W2 = s.W1.to(D), s.W2.to(D)
    in1 = max(0, min(lo + per, n1) - lo)        # elements of the shard that lie in W1
    for q, e in enumerate(at.tolist()):         # the slots get the fresh weights rounded to their type
        fresh = w[e].to(s.W1.dtype).to(D)
        if in1:
            W1[q].view(-1)[lo:lo + in1] = fresh[:in1]
        if in1 < per:
            W2[q].view(-1)[max(lo - n1, 0):lo + per - n1] = fresh[in1:]
    return {"placement": None, "master": w, "m": m, "v": v, "W1": W1, "W2": W2}


def exact(case, seed):
    if 8.0 * case["S"] * 3 * case["d"] * case["f"] > 3e10 and case["kind"] != "router":
        return None         # the slots alone are 30 GB in binary64
    s = prepare(case, seed)
    c, D, kind = s.case, torch.float64, case["kind"]
    if kind == "router":
        X, Wr, dl = s.X.to(D), s.Wr.to(D), s.dlogits.to(D)
        dX = dl @ Wr
        for j in range(c["k"]):
            dX += s.dXp[s.roa.view(-1, c["k"])[:, j].long()].to(D)
        return {"logits": X @ Wr.t() + s.b.to(D), "dWr": dl.t() @ X, "db": dl.sum(0), "dX": dX}
    if kind == "optimizer":
        return _exact_optimizer(s, s.hist.tolist(), s.dW1, s.dW2)
    if kind in ("backward", "slots"):       # what the forward saved is given
        s.rows, s.p = s.hist.tolist(), torch.softmax(s.logits.to(D), 1)
        s.xidx, s.xgate, s.xroa = s.idx.long(), s.gate.to(D), s.roa.view(-1, c["k"]).long()
        s.xXp, s.xUV, s.xH, s.xYp = (t.to(D) for t in (s.Xp, s.UV, s.H, s.Yp))
    if kind == "forward":
        return _exact_forward(s)
    if kind == "backward":
        return _exact_backward(s)
    if kind == "slots":
        dXp, dW1, dW2 = _exact_experts(s, s.dYp.to(D))
        return {"dXp": dXp, "dW1": dW1[s.placement.long()], "dW2": dW2[s.placement.long()]}
    out = _exact_forward(s)
    for n in ("Xp", "UV", "H", "Yp"):
        del out[n]
    back = _exact_backward(s)
    return {**out, **back, **_exact_optimizer(s, s.xhist, back["dW1"], back["dW2"])}
