"""Performance cases of the scenario-batched Split and its screening surrogate.

Each case is one call that a program makes through the package's public entry points, with what
that program has in hand beforehand (context, instance, device demand matrix, captured graph,
trained weights) made by prepare(). Sizes, capacities and demand laws are those of the
repository's workloads (``gen/``, ``bench.py``) or lie between and around them:

  eval      one giant tour over S scenarios (``SplitContext.eval``), from a 20-customer tour over
            1000 scenarios to 1000 customers over 2^20; windows (capacity over mean demand) of a
            few to about a hundred customers; coordinates or a user distance matrix; a demand
            matrix with or without padding between its rows
  batch     tours of uneven length over one scenario matrix (``SplitContext.eval_batch``)
  graph     the neighbours of a search's incumbent, replayed from a captured graph
  predict   the surrogate's predictions of a candidate pool (``SplitNN.predict``)
  gradient  the surrogate's forward and backward pass over a training batch
  topk      the K smallest of C scores (``topk_smallest``)
  screen    predict every candidate, keep 1%, evaluate those exactly (``SplitNN.screen``)
"""
import math

import numpy as np
import torch

import paper_2511_18022_amd as sg

SHIFT, SCALE, LENGTH = 60000.0, 3000.0, 1000.0
WIDTH, TAPS, CI0, FEATURES = 128, 5, 32, 8


def listed():
    return [
        # the smallest call: a short route plan over a first sample of scenarios (launch-bound)
        {"name": "eval-n20-s1000", "kind": "eval", "n": 20, "S": 1000, "law": "uniform",
         "mean": 10.5, "Q": 100, "pad": 0, "matrix": False},
        # a medium instance with short windows (about 13 customers a route)
        {"name": "eval-n200-s100k", "kind": "eval", "n": 200, "S": 100_000, "law": "poisson",
         "mean": 15.0, "Q": 200, "pad": 0, "matrix": False},
        # the smallest scenario count of the runtime-against-scenarios experiment
        {"name": "eval-n1000-s10k", "kind": "eval", "n": 1000, "S": 10_000, "law": "copula",
         "mean": 20.0, "Q": 500, "pad": 0, "matrix": False},
        # its largest, the headline workload
        {"name": "eval-n1000-s1m", "kind": "eval", "n": 1000, "S": 1 << 20, "law": "copula",
         "mean": 20.0, "Q": 500, "pad": 0, "matrix": False},
        # large vehicles (about 60 customers a route), odd sizes, padded rows, a user's matrix
        {"name": "eval-n701-long", "kind": "eval", "n": 701, "S": 20_011, "law": "copula",
         "mean": 20.0, "Q": 1200, "pad": 13, "matrix": True},
        # a search's candidates of uneven length
        {"name": "batch-256", "kind": "batch", "T": 256, "N": 1000, "n_lo": 100, "n_hi": 1000,
         "S": 65_536, "law": "copula", "mean": 20.0, "Q": 500},
        # one iteration of the local search: the neighbours of the incumbent
        {"name": "graph-256x1000", "kind": "graph", "T": 256, "N": 1000, "S": 10_000,
         "law": "copula", "mean": 20.0, "Q": 500},
        # the surrogate over one iteration's pool
        {"name": "predict-4096x1000", "kind": "predict", "T": 4096, "n": 1000},
        # a small pool of short tours
        {"name": "predict-100x203", "kind": "predict", "T": 100, "n": 203},
        # a training batch, forward and backward
        {"name": "gradient-128x1000", "kind": "gradient", "T": 128, "n": 1000},
        # the shortlist of a million candidates
        {"name": "topk-1m", "kind": "topk", "C": 1_000_000, "K": 10_000},
        # screening as a whole
        {"name": "screen-16k", "kind": "screen", "C": 16_384, "n": 1000, "K": 164, "S": 65_536,
         "law": "copula", "mean": 20.0, "Q": 500},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _law(rng):
    """A demand law, its mean and a capacity: windows of 5 to 90 customers."""
    law = rng.choice(["uniform", "poisson", "copula", "copula"])
    mean = {"uniform": 10.5, "poisson": 15.0, "copula": 20.0}[law]
    window = math.exp(rng.uniform(math.log(5.0), math.log(90.0)))
    return law, mean, max(int(round(window * mean)), 2 * int(mean))


def draw(rng):
    kind = rng.choice(["eval"] * 5 + ["batch", "batch", "graph", "predict", "gradient", "topk",
                                      "screen"])
    if kind == "eval":
        law, mean, Q = _law(rng)
        n = _log_int(rng, 12, 2000)
        most = 1_000_000_000 if Q / mean < 30 else 30_000_000
        S = _log_int(rng, 500, max(1000, min(1 << 20, most // n)))
        return {"kind": kind, "n": n, "S": S, "law": law, "mean": mean, "Q": Q,
                "pad": rng.choice([0, 0, 1, 5, 64]), "matrix": n <= 600 and rng.random() < 0.3}
    if kind == "batch":
        law, mean, Q = _law(rng)
        N = _log_int(rng, 60, 1000)
        T = _log_int(rng, 4, 256)
        most = 8_000_000_000 if Q / mean < 30 else 60_000_000
        S = _log_int(rng, 500, max(1000, min(65_536, most // (T * N))))
        return {"kind": kind, "T": T, "N": N, "n_lo": max(1, N // 10), "n_hi": N, "S": S,
                "law": law, "mean": mean, "Q": Q}
    if kind == "graph":
        return {"kind": kind, "T": _log_int(rng, 16, 256), "N": _log_int(rng, 100, 1000),
                "S": _log_int(rng, 1000, 10_000), "law": "copula", "mean": 20.0,
                "Q": rng.randrange(200, 700)}
    if kind == "predict":
        n = _log_int(rng, 20, 1000)
        return {"kind": kind, "T": _log_int(rng, 8, min(4096, 4_096_000 // n)), "n": n}
    if kind == "gradient":
        n = _log_int(rng, 20, 1000)
        return {"kind": kind, "T": _log_int(rng, 4, min(256, 128_000 // n)), "n": n}
    if kind == "topk":
        C = _log_int(rng, 1000, 1_000_000)
        return {"kind": kind, "C": C, "K": max(1, int(C * rng.uniform(0.001, 0.1)))}
    n = _log_int(rng, 60, 1000)
    C = _log_int(rng, 500, 16_384)
    return {"kind": kind, "C": C, "n": n, "K": max(1, C // 100), "S": _log_int(rng, 2000, 65_536),
            "law": "copula", "mean": 20.0, "Q": 500}


# ------------------------------------------------------------------------- inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(1000 + int(seed))


def _coords(g, N):
    return torch.randint(0, 1000, (N + 1, 2), generator=g, device="cuda", dtype=torch.int32)


def _demand(g, N, S, law, mean, Q, pad=0):
    """int16 [N, S + pad]: uniform on 1..2*mean - 1, Poisson with a rate per customer, or a
    Gaussian copula (AR(1) 0.6 along the customer id) with lognormal marginals of CV 0.5."""
    out = torch.zeros((N, S + pad), dtype=torch.int16, device="cuda")
    if law == "uniform":
        out[:, :S] = torch.randint(1, int(2 * mean), (N, S), generator=g, device="cuda",
                                   dtype=torch.int16).clamp_(max=Q)
    elif law == "poisson":
        lam = mean * (1.0 + (torch.rand(N, generator=g, device="cuda") - 0.5) * 4.0 / 3.0)
        for c in range(0, N, 64):
            rows = lam[c:c + 64, None].expand(-1, S).contiguous()
            out[c:c + 64, :S] = torch.poisson(rows, generator=g).clamp_(max=Q).to(torch.int16)
    else:
        s2 = math.log(1.25)
        mu, sd, rho = math.log(mean) - 0.5 * s2, math.sqrt(s2), 0.6
        z = torch.randn(S, generator=g, device="cuda")
        e = torch.empty_like(z)
        for c in range(N):
            if c:
                e.normal_(generator=g)
                z.mul_(rho).add_(e, alpha=math.sqrt(1.0 - rho * rho))
            out[c, :S] = torch.exp(z * sd + mu).round_().clamp_(max=Q).to(torch.int16)
    return out


def _permutation(g, N):
    return (torch.randperm(N, generator=g, device="cuda") + 1).to(torch.int32)


def _short_tour(xy):
    """Customers in vertical strips, up one and down the next: a short tour to start from."""
    strip = xy[1:, 0] // 50
    up = torch.where(strip % 2 == 0, xy[1:, 1], 1000 - xy[1:, 1])
    return (torch.argsort(strip * 4096 + up, stable=True) + 1).to(torch.int32)


def _reversals(g, tours, most):
    """1..most random segment reversals of every row."""
    T, n = tours.shape
    pos = torch.arange(n, device="cuda").expand(T, n)
    count = torch.randint(1, most + 1, (T, 1), generator=g, device="cuda")
    for k in range(most):
        ends = torch.randint(0, n, (T, 2), generator=g, device="cuda").sort(dim=1).values
        lo, hi = ends[:, :1], ends[:, 1:]
        take = (pos >= lo) & (pos <= hi) & (k < count)
        tours = tours.gather(1, torch.where(take, lo + hi - pos, pos))
    return tours.contiguous()


def _neighbours(g, base, T):
    """2-opt reversals and relocations of one tour, in equal shares."""
    n = base.numel()
    pos = torch.arange(n, device="cuda").expand(T, n)
    i = torch.randint(0, n, (T, 1), generator=g, device="cuda")
    j = torch.randint(0, n, (T, 1), generator=g, device="cuda")
    lo, hi = torch.minimum(i, j), torch.maximum(i, j)
    inside = (pos >= lo) & (pos <= hi)
    turned = torch.where(inside, lo + hi - pos, pos)
    moved = torch.where(inside, torch.where(pos == hi, lo, pos + 1), pos)
    two_opt = torch.arange(T, device="cuda")[:, None] % 2 == 0
    return base[torch.where(two_opt, turned, moved)].contiguous()


def _params(g):
    """Weights in the surrogate's flat layout: He-uniform, small biases."""
    def uniform(shape, fan_in):
        a = math.sqrt(6.0 / fan_in)
        return (torch.rand(shape, generator=g, device="cuda") * 2 - 1) * a

    w1 = torch.zeros((TAPS, CI0, WIDTH), device="cuda")
    w1[:, :FEATURES] = uniform((TAPS, FEATURES, WIDTH), TAPS * FEATURES)
    parts = [w1]
    for layer in range(4):
        if layer:
            parts.append(uniform((TAPS, WIDTH, WIDTH), TAPS * WIDTH))
        parts.append(0.05 * torch.randn(WIDTH, generator=g, device="cuda"))
    parts += [uniform((WIDTH, WIDTH), WIDTH), 0.05 * torch.randn(WIDTH, generator=g, device="cuda"),
              uniform((WIDTH,), WIDTH), 0.05 * torch.randn(1, generator=g, device="cuda")]
    return torch.cat([p.reshape(-1) for p in parts])


def _inputs(case, seed):
    """Every input of a case, from the seed alone (no call into the library)."""
    g = _generator(seed)
    kind = case["kind"]
    if kind == "topk":
        return {"scores": SHIFT + SCALE * torch.randn(case["C"], generator=g, device="cuda")}
    if kind == "eval":
        n = case["n"]
        r = {"xy": _coords(g, n), "tour": _permutation(g, n),
             "demand": _demand(g, n, case["S"], case["law"], case["mean"], case["Q"], case["pad"])}
        if case["matrix"]:
            r["dist"] = torch.randint(1, 1500, (n + 1, n + 1), generator=g, device="cuda",
                                      dtype=torch.int32)
        return r
    if kind == "batch":
        N = case["N"]
        xy = _coords(g, N)
        lens = torch.randint(case["n_lo"], case["n_hi"] + 1, (case["T"],), generator=g,
                             device="cuda").tolist()
        return {"xy": xy, "tours": [_permutation(g, N)[:k] for k in lens],
                "demand": _demand(g, N, case["S"], case["law"], case["mean"], case["Q"])}
    if kind == "graph":
        N = case["N"]
        xy = _coords(g, N)
        return {"xy": xy, "tours": list(_neighbours(g, _short_tour(xy), case["T"])),
                "demand": _demand(g, N, case["S"], case["law"], case["mean"], case["Q"])}
    # the surrogate: a 1000-customer instance whose candidates hold n customers
    n = case["n"]
    xy = _coords(g, 1000)
    base = _short_tour(xy)
    base = base[torch.sort(torch.randperm(1000, generator=g, device="cuda")[:n]).values]
    S = case.get("S", 4096)
    r = {"xy": xy, "params": _params(g),
         "demand": _demand(g, 1000, S, "copula", 20.0, 500),
         "tours": _reversals(g, base.expand(case.get("C", case.get("T")), n), 60)}
    if kind == "gradient":
        # costs above the normalization's mean, as when an earlier training set gave it
        z = 2.5 + 0.5 * torch.randn(case["T"], generator=g, device="cuda")
        r["labels"] = SHIFT + SCALE * z
    return r


# ------------------------------------------------------------------------- the calls

def prepare(case, seed):
    kind = case["kind"]
    r = _inputs(case, seed)
    ctx = sg.SplitContext(0)
    s = {"kind": kind, "ctx": ctx, "case": case}
    if kind == "topk":
        return {**s, "scores": r["scores"]}
    if "dist" in r:
        ctx.set_dist(r["dist"].cpu().numpy())
    else:
        ctx.set_coords(r["xy"].cpu().numpy())
    s["demand"] = r["demand"]
    if kind == "eval":
        s["tour"] = r["tour"].cpu().numpy()
        s["demand"] = r["demand"][:, :case["S"]]
    elif kind in ("batch", "graph"):
        s["tours"] = [t.cpu().numpy() for t in r["tours"]]
        if kind == "graph":
            s["graph"] = ctx.graph(case["T"], case["T"] * case["N"], r["demand"], case["Q"])
    else:
        nn = sg.SplitNN(ctx, seed=1, length_scale=LENGTH)
        nn.set_params(r["params"].cpu().numpy())
        nn.set_scenarios(r["demand"], case.get("Q", 500))
        nn.set_norm(SHIFT, SCALE)
        s |= {"nn": nn, "tours": r["tours"], "labels": r.get("labels")}
    return s


def _moments(stats):
    return {"sum": np.array([x.sum for x in stats]), "sumsq": np.array([x.sumsq for x in stats]),
            "mean": np.array([x.mean for x in stats]), "var": np.array([x.var for x in stats])}


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "eval":
        cost, st = state["ctx"].eval(state["tour"], state["demand"], case["Q"])
        return {"cost": cost, "sum": st.sum, "sumsq": st.sumsq, "mean": st.mean, "var": st.var}
    if kind == "batch":
        cost, stats, _ = state["ctx"].eval_batch(state["tours"], state["demand"], case["Q"])
        return {"cost": cost, **_moments(stats)}
    if kind == "graph":
        cost = state["graph"].launch(state["tours"])
        stats, _ = state["graph"].stats()
        return {"cost": cost, **_moments(stats)}
    if kind == "predict":
        return {"pred": state["nn"].predict(state["tours"])}
    if kind == "gradient":
        grad, loss = state["nn"].gradient(state["tours"], state["labels"])
        return {"grad": grad, "loss": loss}
    if kind == "topk":
        return {"idx": sg.topk_smallest(state["ctx"], state["scores"], case["K"])}
    res = state["nn"].screen(state["tours"], case["K"], state["demand"], case["Q"])
    return {k: res[k] for k in ("pred", "short_idx", "short_mean", "best_idx", "best_mean")}


# ------------------------------------------------------------------------- work

def _net_flops(n):
    """Multiply-adds of the four layers over n positions, two operations each."""
    return 2.0 * n * WIDTH * (TAPS * FEATURES + 3 * TAPS * WIDTH)


def work(case):
    """Bytes: each input once, each output once. Operations: integer operations of the Split at
    six a state (prefix sum, window test, two adds and two minima of a sliding-window minimum),
    multiply-adds of the network's layers at two."""
    kind = case["kind"]
    if kind == "topk":
        return {"bytes": 4.0 * case["C"] + 4.0 * case["K"], "flops": float(case["C"])}
    if kind == "eval":
        return {"bytes": (2.0 * case["n"] + 4.0) * case["S"], "flops": 6.0 * case["n"] * case["S"]}
    if kind in ("batch", "graph"):
        mean_n = case["N"] if kind == "graph" else 0.5 * (case["n_lo"] + case["n_hi"])
        return {"bytes": (2.0 * case["N"] + 4.0 * case["T"]) * case["S"],
                "flops": 6.0 * mean_n * case["T"] * case["S"]}
    weights = 4.0 * (TAPS * FEATURES + 3 * TAPS * WIDTH + WIDTH) * WIDTH
    if kind == "predict":
        T, n = case["T"], case["n"]
        return {"bytes": 4.0 * T * n + 4.0 * T + weights, "flops": T * _net_flops(n)}
    if kind == "gradient":
        T, n = case["T"], case["n"]
        back = 2.0 * n * WIDTH * (3 * TAPS * WIDTH)  # the data gradients of layers 2..4
        return {"bytes": 4.0 * T * n + 4.0 * T + 2 * weights,
                "flops": T * (2 * _net_flops(n) + back)}
    C, n, K, S = case["C"], case["n"], case["K"], case["S"]
    return {"bytes": 4.0 * C * n + 4.0 * C + weights + 2.0 * 1000 * S,
            "flops": C * _net_flops(n) + 6.0 * K * n * S}


# ------------------------------------------------------------------------- reference values

def _distances(r):
    if "dist" in r:
        return r["dist"].to(torch.int64)
    xy = r["xy"].to(torch.int64)
    m = ((xy[:, None] - xy[None]) ** 2).sum(-1)
    k = torch.floor(torch.sqrt(m.double())).to(torch.int64)
    k = torch.where(k * k > m, k - 1, k)
    k = torch.where((k + 1) * (k + 1) <= m, k + 1, k)
    return torch.where(m - k * k > k, k + 1, k)


def _split_costs(tours, d, demand, Q, mean):
    """f(n) [T, S] of tours sorted by falling length, by the recurrence over a window of
    predecessors: f(i) = min over feasible p of f(p) + cost of the route p+1..i."""
    S = demand.shape[1]
    T = len(tours)
    lens = [t.numel() for t in tours]
    wide = min(lens[0], int(3.0 * Q / mean) + 12)
    big = 1 << 29
    P = torch.zeros((wide, T, S), dtype=torch.int32, device="cuda")
    G = torch.full((wide, T, S), big, dtype=torch.int32, device="cuda")
    out = torch.zeros((T, S), dtype=torch.int32, device="cuda")
    ids = torch.zeros((T, lens[0] + 1), dtype=torch.int64, device="cuda")
    for t, tour in enumerate(tours):
        ids[t, :lens[t]] = tour.to(torch.int64)
    arcs = d[ids[:, :-1], ids[:, 1:]]  # past a tour's end: not used
    first, last = d[0, ids], d[ids, 0]
    total = torch.zeros(T, dtype=torch.int64, device="cuda")  # arcs up to the current position
    G[0] = first[:, 0].to(torch.int32)[:, None]  # f(p) + c(0, next) - arcs up to next
    load = torch.zeros((T, S), dtype=torch.int32, device="cuda")
    clipped = torch.zeros((), dtype=torch.bool, device="cuda")
    for i in range(1, lens[0] + 1):
        live = sum(1 for k in lens if k >= i)
        load[:live] += demand[ids[:live, i - 1] - 1].to(torch.int32)
        w = min(i, wide)
        fits = load[None, :live] - P[:w, :live] <= Q
        f = torch.where(fits, G[:w, :live], big).amin(0)
        if i > wide:
            clipped |= fits[i % wide].any()
        base = total[:live] + last[:live, i - 1]
        f = f + base.to(torch.int32)[:, None]
        for t in range(live):
            if lens[t] == i:
                out[t] = f[t]
        if i < lens[0]:
            total += arcs[:, i - 1]
            P[i % wide] = load
            step = (first[:live, i] - total[:live]).to(torch.int32)
            G[i % wide, :live] = f + step[:, None]
    # the oldest predecessor kept was out of reach everywhere: no window was cut short
    if bool(clipped):
        raise ValueError("a window is longer than the reference keeps")
    return out


def _exact_moments(costs):
    mean, var = [], []
    for c in costs.to(torch.int64):
        S, total, square = c.numel(), int(c.sum()), int((c * c).sum())
        mean.append(total / S)
        var.append((S * square - total * total) / S / (S - 1) if S > 1 else 0.0)
    return np.array(mean), np.array(var)


def _features(r, tours, Q):
    xy = r["xy"].double()
    d = _distances(r).double()
    q = r["demand"].double()
    mu = q.mean(1)
    sd = (q.square().mean(1) - mu * mu).clamp_(min=0).sqrt()
    t = tours.to(torch.int64)
    depot = torch.zeros_like(t[:, :1])
    before, after = torch.cat([depot, t[:, :-1]], 1), torch.cat([t[:, 1:], depot], 1)
    return torch.stack([(xy[t, 0] - xy[0, 0]) / LENGTH, (xy[t, 1] - xy[0, 1]) / LENGTH,
                        mu[t - 1] / Q, sd[t - 1] / Q, d[before, t] / LENGTH, d[t, after] / LENGTH,
                        d[0, t] / LENGTH, torch.ones(t.shape, dtype=torch.float64, device="cuda")],
                       dim=-1)


def _unpack(p):
    at = 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return p[at - n:at].reshape(shape)

    layers = []
    for layer in range(4):
        w = take(TAPS, WIDTH if layer else CI0, WIDTH)
        layers.append((w if layer else w[:, :FEATURES], take(WIDTH)))
    return layers, take(WIDTH, WIDTH), take(WIDTH), take(WIDTH), take(1)


def _network(p, x):
    """The network in 64 bits: x [T, n, 8] to y [T]."""
    layers, wa, ba, wb, bb = _unpack(p)
    T, n, _ = x.shape
    for w, b in layers:
        ci = w.shape[1]
        padded = torch.nn.functional.pad(x, (0, 0, 2, 2))
        spans = torch.cat([padded[:, k:k + n] for k in range(TAPS)], -1).reshape(T * n, TAPS * ci)
        x = torch.relu(spans @ w.reshape(TAPS * ci, WIDTH) + b).reshape(T, n, WIDTH)
    z = x.mean(1)
    return torch.relu(z @ wa.t() + ba) @ wb + bb


def exact(case, seed):
    kind = case["kind"]
    if kind == "topk":
        return None
    r = _inputs(case, seed)
    if kind in ("eval", "batch", "graph"):
        d = _distances(r)
        S = case["S"]
        tours = [r["tour"]] if kind == "eval" else r["tours"]
        order = sorted(range(len(tours)), key=lambda t: -tours[t].numel())
        mean, var = np.zeros(len(tours)), np.zeros(len(tours))
        room = max(1, int(5e8 // (S * min(tours[order[0]].numel(), 3.0 * case["Q"] / case["mean"] + 12))))
        for k in range(0, len(order), room):
            part = order[k:k + room]
            costs = _split_costs([tours[t] for t in part], d, r["demand"][:, :S], case["Q"],
                                 case["mean"])
            mean[part], var[part] = _exact_moments(costs)
        none = {"cost": None, "sum": None, "sumsq": None}
        return {**none, "mean": mean, "var": var} if kind != "eval" else \
            {**none, "mean": float(mean[0]), "var": float(var[0])}
    p = r["params"].double()
    Q = case.get("Q", 500)
    T, n = r["tours"].shape
    room = max(1, 64_000 // n)
    if kind == "gradient":
        p.requires_grad_(True)
        y_hat = (r["labels"].double() - SHIFT) / SCALE
        loss = 0.0
        for k in range(0, T, room):
            y = _network(p, _features(r, r["tours"][k:k + room], Q))
            part = ((y - y_hat[k:k + room]) ** 2).sum() / T
            part.backward()
            loss += float(part)
        return {"grad": p.grad, "loss": loss}
    with torch.no_grad():
        pred = torch.cat([_network(p, _features(r, r["tours"][k:k + room], Q)) * SCALE + SHIFT
                          for k in range(0, T, room)])
    if kind == "predict":
        return {"pred": pred}
    return {"pred": pred, "short_idx": None, "short_mean": None, "best_idx": None,
            "best_mean": None}
