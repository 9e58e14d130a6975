"""Workloads of the progressive approximate LSTM for performance measurement.

Each case is one call (or one chain of calls) that a program makes through the
public binding: a run of one sequence or several at one budget or several, a
run with a budget per timestep, stacked layers, the bf16 batched run, the
exact baseline and the device factorisation.  Sizes are those of the named
synthetic workloads (``paper_1905_00689_amd.synth``), with ranks that keep the
factorisation short where the budget measured does not need the whole rank.

``prepare`` factorises the weights (the handle a program keeps) and places the
inputs on the GPU; ``run`` is the call alone.  ``exact`` evaluates Eq. (1) and
the cell update in float64 on the factor lists the model holds (what the run
is given; the greedy chain behind them is numerically chaotic past a few dozen
terms, so no second factorisation could stand in for them), or the dense LSTM
on the weights, or, for the factorisation itself, a float64 chain of its own.
"""

import math

import numpy as np
import torch

from paper_1905_00689_amd import binding as B
from paper_1905_00689_amd import synth


def listed():
    return [
        # the smallest model: a sensor-sized LSTM on a short window, four
        # budgets of it in one call; launches and latency are all there is
        dict(name="tiny", op="run", D=64, H=32, T=8, B=1, K="1,4,16,96", rank=96, p=0.5, weights="gauss"),
        # the paper's model (8256 CNN features, 64 units, 100 frames) at a
        # coarse budget, where approximation pays most
        dict(name="paper", op="run", D=8256, H=64, T=100, B=1, K="16", rank=16, nz=130, weights="decay"),
        # the driving workload at its full budget: the headline figure
        dict(name="driving", op="run", D=2048, H=512, T=16, B=1, K="512", rank=512, p=0.75, weights="gauss"),
        # one driving sequence, refined at four budgets in one call
        dict(name="levels", op="run", D=2048, H=512, T=16, B=1, K="16,64,128,192", rank=192, p=0.75,
             weights="gauss"),
        # eight cameras at once: sequences that continue (h0, c0 in, c out)
        dict(name="sequences", op="run", D=2048, H=512, T=16, B=8, K="128", rank=128, p=0.75, weights="gauss",
             state=True),
        # a budget per timestep over a longer clip (the time left varies)
        dict(name="schedule", op="schedule", D=2048, H=512, T=64, B=1, K="128", rank=128, p=0.75, weights="gauss"),
        # two stacked layers of 1024 units on wide features, one sequence
        dict(name="stack", op="stack", D=4096, H=1024, T=32, B=1, K="64,64", rank=64, p=0.75, weights="gauss"),
        # the widest layer, eight sequences of 64 steps, heavy pruning
        dict(name="deadline", op="run", D=2048, H=2048, T=64, B=8, K="64", rank=64, p=0.9, weights="gauss"),
        # throughput serving: 256 sequences on the bf16 matrix path
        dict(name="batched", op="batched", D=2048, H=512, T=16, B=256, K="512", rank=512, p=0.75, weights="gauss"),
        # the exact LSTM that outputs are compared with, at the driving shape
        dict(name="exact", op="exact", D=2048, H=512, T=16, B=1, weights="gauss"),
        # and at the widest layer with eight sequences: the largest call
        dict(name="exact wide", op="exact", D=2048, H=2048, T=64, B=8, weights="gauss"),
        # factorising a small layer on the device (a model is prepared once,
        # but a program that adapts one waits for it)
        dict(name="prepare", op="prepare", D=512, H=256, T=1, B=1, rank=16, p=0.75, weights="gauss"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["run", "run", "levels", "sequences", "schedule", "stack", "batched", "batched", "exact", "rows",
                     "prepare"])
    D, H, T = _log(rng, 48, 4096), _log(rng, 24, 1024), _log(rng, 6, 80)
    p = rng.choice([0.0, 0.5, 0.75, 0.9])
    c = dict(op=op, D=D, H=H, T=T, B=1, p=p, weights="gauss")
    if op in ("run", "levels", "sequences"):
        c["op"] = "run"
        c["K"] = str(_log(rng, 1, 144))
        c["state"] = rng.random() < 0.5
        c["groups"] = rng.choice([4, 4, 4, 1])
        if op == "levels":
            c["K"] = ",".join(str(_log(rng, 1, 96)) for _ in range(rng.randint(2, 5)))
        if op == "sequences":
            c["B"] = rng.randint(2, 8)
    elif op == "schedule":
        c["K"], c["B"] = str(_log(rng, 2, 96)), rng.choice([1, 1, 2, 4])
    elif op == "stack":
        c["K"] = "%d,%d" % (_log(rng, 1, 64), _log(rng, 1, 64))
    elif op == "batched":
        c.update(D=_log(rng, 64, 2048), H=_log(rng, 32, 512), T=_log(rng, 6, 24), B=_log(rng, 17, 256),
                 K=str(_log(rng, 4, 128)), p=rng.choice([0.5, 0.75, 0.9]), state=rng.random() < 0.5)
    elif op in ("exact", "rows"):
        c.update(B=rng.choice([1, 1, 2, 3, 5, 8]), state=rng.random() < 0.5)
        del c["p"]
        if op == "rows":
            c["rows"] = rng.randint(1, H)
    else:
        c.update(D=_log(rng, 48, 1024), H=_log(rng, 48, 384), T=1, rank=rng.randint(6, 16))
    if "K" in c:
        c["rank"] = max(int(k) for k in c["K"].split(","))
    return c


def _budgets(case):
    return [int(k) for k in case["K"].split(",")]


def _nz(case, C):
    return case["nz"] if "nz" in case else C - int(math.floor(case["p"] * C))


def _dims(case):
    """Input widths of the layers (one, or two for a stack)."""
    return [case["D"], case["H"]] if case["op"] == "stack" else [case["D"]]


def _weights(case, seed):
    """[(W_ih, W_hh, b)] host float32 per layer: N(0, 1/sqrt(D+H)) weights, or
    decaying spectra and column weights as a trained model shows."""
    out, H = [], case["H"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    for i, D in enumerate(_dims(case)):
        if case["weights"] == "decay":
            W, b = synth.lstm_weights_decay(np.random.default_rng([seed, i]), D, H)
            out.append((np.ascontiguousarray(W[:, :D]), np.ascontiguousarray(W[:, D:]), b))
        else:
            sd = 1.0 / math.sqrt(D + H)
            wi = torch.randn(4 * H, D, generator=g, device="cuda").mul_(sd)
            wh = torch.randn(4 * H, H, generator=g, device="cuda").mul_(sd)
            b = torch.randn(4 * H, generator=g, device="cuda").mul_(0.1)
            out.append((wi.cpu().numpy(), wh.cpu().numpy(), b.cpu().numpy()))
    return out


def _inputs(case, seed):
    """x [T, B, D], half of it zeros as after a rectifier, and the state of a
    sequence that continues (h0, c0, or None)."""
    g = torch.Generator(device="cuda").manual_seed(seed + (1 << 32))
    T, Bn, D, H = case["T"], case["B"], case["D"], case["H"]
    x = torch.randn(T, Bn, D, generator=g, device="cuda").clamp_(min=0.0)
    h0 = c0 = None
    if case.get("state"):
        h0 = torch.randn(Bn, H, generator=g, device="cuda").mul_(0.4).tanh_()
        c0 = torch.randn(Bn, H, generator=g, device="cuda").mul_(0.5)
    return x, h0, c0


def _schedule(case, seed):
    """K_t over 0 .. the case's budget, a third of the steps cut short."""
    r = np.random.default_rng([seed, 3])
    k = int(case["K"])
    full = r.random(case["T"]) > 0.33
    return np.where(full, k, r.integers(0, k + 1, case["T"])).astype(np.int32)


def _factorise(case, wi, wh, b):
    H, D = case["H"], wi.shape[1]
    kw = dict(nz=case["nz"]) if "nz" in case else dict(prune_ratio=case["p"])
    return B.approx_lstm_prepare(wi, wh, b, D, H, case["rank"], groups=case.get("groups", 4),
                                 factor_dtype=1 if case["op"] == "batched" else 0,
                                 flags=B.FLAG_DEVICE_FACTORISE, **kw)


def prepare(case, seed):
    T, Bn, H, op = case["T"], case["B"], case["H"], case["op"]
    layers = _weights(case, seed)
    s = dict(case=case, weights=layers)
    if op == "prepare":
        return s
    s["x"], s["h0"], s["c0"] = _inputs(case, seed)
    if op in ("exact", "rows"):
        s["model"] = B.approx_lstm_exact_prepare(*layers[0], case["D"], H)
        s["h"] = torch.empty(T, Bn, H, device="cuda")
        s["c"] = torch.empty(Bn, H, device="cuda")
    else:
        s["models"] = [_factorise(case, *w) for w in layers]
        n = 1 if op in ("schedule", "stack") else len(_budgets(case))
        s["h"] = torch.empty(*([T, Bn, H] if op == "schedule" else [n, T, Bn, H]), device="cuda")
        s["c"] = torch.empty(*([Bn, H] if op == "schedule" else [n, Bn, H]), device="cuda")
        s["k"] = _schedule(case, seed) if op == "schedule" else _budgets(case)
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "prepare":
        m = _factorise(case, *s["weights"][0])
        return [B.approx_lstm_get_factors(m, g) for g in range(4)]
    if op == "exact":
        B.approx_lstm_exact_run(s["model"], s["x"], s["h"], s["h0"], s["c0"], s["c"])
    elif op == "rows":
        B.approx_lstm_exact_run_rows(s["model"], s["x"], case["rows"], s["h"], s["h0"], s["c0"], s["c"])
    elif op == "schedule":
        B.approx_lstm_run_schedule(s["models"][0], s["x"], s["k"], s["h"], s["h0"], s["c0"], s["c"])
    elif op == "stack":
        B.approx_lstm_run_stack(s["models"], s["x"], [s["k"]], s["h"])
        return s["h"]
    else:
        B.approx_lstm_run(s["models"][0], s["x"], s["k"], s["h"], s["h0"], s["c0"], s["c"])
    return [s["h"], s["c"]]


def work(case):
    T, Bn, H, op = case["T"], case["B"], case["H"], case["op"]
    G = case.get("groups", 4)
    if op == "prepare":
        # every term needs one pass over the residual for its update and, at
        # the least, one product with it
        C, n = case["D"] + H, case["rank"]
        return dict(bytes=4.0 * 4 * H * C + 4.0 * n * (1 + H + 2 * _nz(case, C)) * 4, flops=4.0 * n * 4 * H * C)
    xb, hb = 4.0 * T * Bn * case["D"], 4.0 * T * Bn * H
    if op in ("exact", "rows"):
        C, R = case["D"] + H, 4 * case.get("rows", H)
        return dict(bytes=4.0 * R * C + 16.0 * H + xb + hb, flops=2.0 * R * C * T * Bn)
    by = fl = 0.0
    ks = _budgets(case)
    val, idx = (2, 2) if op == "batched" else (4, 2)
    for i, D in enumerate(_dims(case)):
        nz, rg = _nz(case, D + H), 4 * H // G
        if op == "schedule":
            k = kf = int(case["K"])
        elif op == "stack":
            k = kf = ks[i]
        else:
            k, kf = max(ks), sum(ks)
        by += G * k * (val * rg + (val + idx) * nz + 4.0) + 16.0 * H
        fl += G * kf * (2.0 * nz + 2.0 * rg + 1) * T * Bn
    return dict(bytes=by + xb + hb * (len(ks) if op == "run" else 1), flops=fl)


def tolerance(case):
    # measured against exact(): fp32 runs 2e-7 to 6e-7, the bf16 run 2e-3
    # (x, h and z are rounded to bf16), stored factors 3e-8 (fp32 rounding)
    if case["op"] == "batched":
        return {"rel": 4e-3, "max": 6e-2}
    if case["op"] == "prepare":
        return {"rel": 1e-6, "max": 1e-4, "differ": 1e-3}
    return {"rel": 5e-6, "max": 2e-4}


# ---- float64 references


def _lists(m, G):
    """The factor lists a run is given: sigma [G, N], U [G, Rg, N], V dense [G, N, C], float64 on the GPU."""
    C = m.info["aug_size"]
    sig, U, V = [], [], []
    for g in range(G):
        f = B.approx_lstm_get_factors(m, g)
        v = torch.zeros(f["sigma"].shape[0], C, dtype=torch.float64, device="cuda")
        v.scatter_(1, torch.from_numpy(f["v_idx"].astype(np.int64)).cuda(), torch.from_numpy(f["v_val"]).cuda().double())
        sig.append(torch.from_numpy(f["sigma"]).cuda().double())
        U.append(torch.from_numpy(f["u"]).cuda().double().t().contiguous())
        V.append(v)
    return torch.stack(sig), torch.stack(U), torch.stack(V)


def _cell(y, c, H):
    i, f, g, o = y[:, :H], y[:, H:2 * H], y[:, 2 * H:3 * H], y[:, 3 * H:]
    c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(g)
    return torch.sigmoid(o) * torch.tanh(c), c


def _start(case, h0, c0):
    z = torch.zeros(case["B"], case["H"], dtype=torch.float64, device="cuda")
    return (z if h0 is None else h0.double()), (z if c0 is None else c0.double())


def _progressive(case, lists, b, x, ks, h0, c0):
    """One level: x [T, B, D] float64, ks the budget of every timestep."""
    sig, U, V = lists
    G, H, D = sig.shape[0], case["H"], x.shape[2]
    h, c = _start(case, h0, c0)
    hs = []
    for t in range(x.shape[0]):
        k = int(ks[t])
        xh = torch.cat([x[t], h], 1)
        y = [(U[g, :, :k] @ (sig[g, :k, None] * (V[g, :k, :D + H] @ xh.t()))).t() for g in range(G)]
        h, c = _cell(torch.cat(y, 1) + b, c, H)
        hs.append(h)
    return torch.stack(hs), c


def _chain(case, wi, wh):
    """The factorisation of each gate in float64: top triplet of the residual
    (largest entry of v positive), prune v to its NZ largest, deflate."""
    H, C = case["H"], case["D"] + case["H"]
    nz, out = _nz(case, C), []
    W = torch.cat([torch.from_numpy(wi), torch.from_numpy(wh)], 1).cuda().double()
    for g in range(4):
        R = W[g * H:(g + 1) * H].clone()
        f = dict(sigma=[], u=[], v_idx=[], v_val=[])
        for _ in range(case["rank"]):
            if H <= C:
                u = torch.linalg.eigh(R @ R.t())[1][:, -1]
            else:
                v = torch.linalg.eigh(R.t() @ R)[1][:, -1]
                u = R @ v
                u = u / u.norm()
            v = R.t() @ u
            s = v.norm()
            v = v / s
            sign = torch.sign(v[v.abs().argmax()])
            u, v = u * sign, v * sign
            idx = torch.sort(torch.argsort(v.abs(), descending=True, stable=True)[:nz])[0]
            kept = torch.zeros_like(v)
            kept[idx] = v[idx]
            R -= s * torch.outer(u, kept)
            for name, t in (("sigma", s), ("u", u), ("v_idx", idx), ("v_val", v[idx])):
                f[name].append(t.cpu())
        out.append({k: torch.stack(t).numpy() for k, t in f.items()})
    return out


def exact(case, seed):
    H, op = case["H"], case["op"]
    layers = _weights(case, seed)
    if op == "prepare":
        return _chain(case, *layers[0][:2])
    x, h0, c0 = _inputs(case, seed)
    xd = x.double()
    if op in ("exact", "rows"):
        wi, wh, b = (torch.from_numpy(a).cuda().double() for a in layers[0])
        if op == "rows":
            dead = (torch.arange(4 * H, device="cuda") % H) >= case["rows"]
            wi[dead] = 0.0
            wh[dead] = 0.0
        h, c = _start(case, h0, c0)
        hs = []
        for t in range(case["T"]):
            h, c = _cell(xd[t] @ wi.t() + h @ wh.t() + b, c, H)
            hs.append(h)
        return [torch.stack(hs), c]
    G = case.get("groups", 4)
    lists = [_lists(_factorise(case, *w), G) for w in layers]
    bs = [torch.from_numpy(w[2]).cuda().double() for w in layers]
    T = case["T"]
    if op == "schedule":
        return list(_progressive(case, lists[0], bs[0], xd, _schedule(case, seed), h0, c0))
    if op == "stack":
        for f, b, k in zip(lists, bs, _budgets(case)):
            xd = _progressive(case, f, b, xd, [k] * T, None, None)[0]
        return xd[None]
    outs = [_progressive(case, lists[0], bs[0], xd, [k] * T, h0, c0) for k in _budgets(case)]
    return [torch.stack([h for h, _ in outs]), torch.stack([c for _, c in outs])]
