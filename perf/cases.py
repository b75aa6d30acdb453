"""Performance cases of the framework: what its users have it do, by size.

Each case is one pass through the public entry points (`Planner`, `Network`,
`optimize_many`), as a planning program calls them:

* evaluate      objective and gradient of a weight batch at given dwell weights, on
                device arrays (`evaluate_noalloc`) or host arrays (`evaluate`);
* plan          a weight batch from its start to finished plans: `set_weights`, the
                stages of `optimize`, `dwell_times`, and, where asked, `metrics` and
                `select_plan`;
* batch         several uneven cases in lockstep (`optimize_many`);
* quality       `metrics` and `select_plan` of finished plans;
* patient       a new patient on a running planner: `load_case`, `set_weights`, the
                first evaluation;
* train         Adam steps of the learned warm start's network.

Geometry, weights and sizes are those of the repository's synthetic cases: a target
ellipsoid, the urethra, bladder and rectum slabs, catheters on a 1 cm grid, hidden
weights log-uniform in [0.1, 10].  Sizes follow the paper's cohort (102 to 385 dwells,
2,753 to 15,998 points), the benchmark (360 x 20,000 x 1,000 plans) and its uneven batch
(120 to 400 dwells, 8,000 to 30,000 points).
"""
import math

import numpy as np
import torch

from paper_1904_01567_amd import Network, Planner, class_solution, optimize_many

DEVICE = "cuda:0"
RX = 15.0
SPLIT = (0.5, 0.1, 0.2, 0.2)  # points per structure: target, urethra, bladder, rectum
# surface and volume groups: share of the points, organ of each group
SV_SPLIT = (0.1, 0.4, 0.05, 0.05, 0.05, 0.15, 0.05, 0.15)
SV_ORGAN = np.array([0, 0, 1, 1, 2, 2, 3, 3], dtype=np.int32)


def listed():
    return [
        # the repository's small case (16 catheters x 10 dwells, 8 plans): the smallest
        # call, one evaluation on device arrays, where launches and latency count
        dict(name="evaluate small", kind="evaluate", K=160, M=2400, P=8, dtype="f32acc64", arrays="device"),
        # one plan of the paper-scale case (the first point of the plan-count scaling)
        dict(name="evaluate one plan", kind="evaluate", K=360, M=20000, P=1, dtype="f32", arrays="device"),
        # the paper-scale batch in BF16, the arithmetic of the first optimiser steps
        dict(name="evaluate bf16", kind="evaluate", K=360, M=20000, P=1000, dtype="bf16", arrays="device"),
        # the same batch with the FP64-accumulated dose, called with host arrays
        dict(name="evaluate acc64 host", kind="evaluate", K=360, M=20000, P=1000, dtype="f32acc64", arrays="host"),
        # odd sizes in FP8: dwells and points off every tile, a part-filled plan tile
        dict(name="evaluate fp8 ragged", kind="evaluate", K=277, M=12347, P=333, dtype="fp8", arrays="device"),
        # a few plans of the small case to a fixed step count: rounds bound by latency
        dict(name="plan small", kind="plan", K=160, M=2400, P=8, dtype="f32acc64", stages="f32acc64:60", eps=0.0,
             finish=False, evaluations=63.0),
        # the largest clinical layout at the clinical stop rule, to metrics and selection
        dict(name="plan clinical", kind="plan", K=385, M=15998, P=1000, dtype="f32acc64",
             stages="f32acc64:2000", eps=1e-3, finish=True, evaluations=75.0),
        # the benchmark's own run: 1,000 plans, precision ladder, to its stop threshold
        dict(name="plan ladder", kind="plan", K=360, M=20000, P=1000, dtype="bf16",
             stages="bf16:100,f32:500,f32acc64:2000", eps=2e-10, finish=False, evaluations=1500.0),
        # uneven cases in grouped lockstep rounds replayed from a graph
        dict(name="batch uneven", kind="batch", n=8, K0=120, K1=400, M0=8000, M1=30000, P=250, dtype="f32",
             stages="f32:50", eps=0.0, evaluations=53.0),
        # plan quality with surface and volume groups and a five times denser DVH point set
        dict(name="quality dvh", kind="quality", K=360, M=20000, Md=100000, P=1000),
        # the next patient arrives: case upload, dose-rate matrix, first evaluation
        dict(name="patient bf16", kind="patient", K=360, M=20000, P=1000, dtype="bf16"),
        # training of the warm start's network at its own layout and batch
        dict(name="train", kind="train", n_in=68, hidden=256, depth=3, n_out=360, B=1024, rows=8192, steps=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evaluate", "evaluate", "evaluate", "plan", "plan", "batch", "quality", "quality", "patient",
                       "patient", "train"])
    K = rng.randint(102, 400)
    M = _log_int(rng, 2400, 30000)
    P = _log_int(rng, 1, 1000)
    if kind == "evaluate":
        return dict(kind=kind, K=K, M=M, P=P, dtype=rng.choice(["f32", "bf16", "fp8", "f32acc64"]),
                    arrays=rng.choice(["device", "device", "host"]))
    if kind == "plan":
        if rng.random() < 0.5:
            n = rng.randint(10, 60)
            return dict(kind=kind, K=K, M=M, P=P, dtype="f32acc64", stages="f32acc64:%d" % n, eps=0.0, finish=False,
                        evaluations=1.05 * n)
        return dict(kind=kind, K=K, M=min(M, 20000), P=P, dtype="bf16", stages="bf16:50,f32:100,f32acc64:2000",
                    eps=1e-3, finish=True, evaluations=75.0)
    if kind == "batch":
        n = rng.randint(2, 8)
        steps = rng.randint(10, 50)
        return dict(kind=kind, n=n, K0=120, K1=400, M0=8000, M1=30000, P=_log_int(rng, 8, 250), dtype="f32",
                    stages="f32:%d" % steps, eps=0.0, evaluations=1.05 * steps)
    if kind == "quality":
        return dict(kind=kind, K=K, M=min(M, 20000), Md=rng.choice([0, 5]) * min(M, 20000), P=P)
    if kind == "patient":
        return dict(kind=kind, K=K, M=M, P=P, dtype=rng.choice(["f32", "bf16", "fp8", "f32acc64"]))
    return dict(kind=kind, n_in=68, hidden=_log_int(rng, 64, 256), depth=rng.randint(1, 3), n_out=K,
                B=_log_int(rng, 32, 1024), rows=2048, steps=rng.randint(5, 20))


# ---- inputs ----

def _ball(r, n, d):
    v = r.normal(size=(n, d))
    v *= (r.uniform(size=(n, 1)) ** (1.0 / d)) / np.linalg.norm(v, axis=1, keepdims=True)
    return v


def _points(r, n, organ, surface, a):
    """n points of one organ, inside it or on its surface."""
    if organ == 0:
        v = _ball(r, n, 3)
        return (v / np.linalg.norm(v, axis=1, keepdims=True) if surface else v) * a
    if organ == 1:
        ang, z = r.uniform(0, 2 * math.pi, n), r.uniform(-a[2], a[2], n)
        rad = 0.3 if surface else 0.3 * np.sqrt(r.uniform(size=n))
        return np.stack([rad * np.cos(ang), rad * np.sin(ang), z], 1)
    v = _ball(r, n, 2)
    near = r.uniform(size=n) * 0.5
    if surface:
        near = np.where(near < 0.25, 0.0, 0.5)
    y = (a[1] + 0.5 + near) * (1.0 if organ == 2 else -1.0)
    return np.stack([v[:, 0] * a[0], y, v[:, 1] * a[2]], 1)


def _shares(n, parts):
    c = [int(n * p) for p in parts[1:]]
    return [n - sum(c)] + c


def _geometry(seed, K, M, Md=None):
    """One synthetic patient as load_case takes it (keyword arguments)."""
    r = np.random.default_rng(seed)
    a = np.array([2.0, 1.75, 1.75]) * r.uniform(0.9, 1.1, 3)
    per = 20 if K >= 40 else 4
    n_cath = max(1, -(-K // per))
    span = int(math.ceil(math.sqrt(n_cath))) + 2
    nodes = sorted((x * x + y * y, math.atan2(y, x) % (2 * math.pi), x, y)
                   for x in np.arange(-span, span) + 0.5 for y in np.arange(-span, span) + 0.5)[:n_cath]
    z = (np.arange(per) - (per - 1) / 2.0) * (5.0 / per) * a[2] / 1.75
    dwell = np.array([[n[2], n[3], v] for n in nodes for v in z])[:K]
    sv = Md is not None
    parts = SV_SPLIT if sv else SPLIT
    counts = _shares(M, parts)
    organ = SV_ORGAN if sv else np.arange(4, dtype=np.int32)
    pts = np.concatenate([_points(r, n, organ[g], sv and g % 2 == 0, a) for g, n in enumerate(counts)])
    group = np.repeat(np.arange(len(parts), dtype=np.int32), counts)
    slab = 0.5 * math.pi * a[0] * a[2]
    vol = np.array([4.0 / 3.0 * math.pi * a[0] * a[1] * a[2], math.pi * 0.09 * 2 * a[2], slab, slab])
    rows = class_solution.SURFACE_VOLUME if sv else class_solution.VOLUME
    kw = dict(dwell_xyz=dwell, point_xyz=pts, group=group, group_params=rows, volume_cc=vol, prescription_gy=RX,
              target_group=0)
    if sv:
        kw["group_organ"] = SV_ORGAN
        if Md > 0:
            dc = _shares(Md, SPLIT)
            kw["dvh_xyz"] = np.concatenate([_points(r, n, j, False, a) for j, n in enumerate(dc)])
            kw["dvh_organ"] = np.repeat(np.arange(4, dtype=np.int32), dc)
    return kw


def _weights(seed, P):
    w = np.exp(np.random.default_rng(seed).uniform(math.log(0.1), math.log(10.0), size=(P, 4)))
    return w / w.sum(1, keepdims=True)


def _dose_rate(dwell, pts):
    """Dose-rate matrix in 64 bits on the device: (1 - 0.01 r) / max(r, 0.1 cm)^2."""
    d, p = (torch.tensor(v, dtype=torch.float64, device=DEVICE) for v in (dwell, pts))
    r = ((p[:, None, :] - d[None, :, :]) ** 2).sum(2).sqrt()
    return (1.0 - 0.01 * r) / r.clamp(min=0.1) ** 2


def _start_time(kw, D):
    organ = kw.get("group_organ", np.arange(8, dtype=np.int32))[kw["group"]]
    rows = D[torch.tensor(organ == 0, device=DEVICE)]
    return RX / float(rows.sum(1).mean())


def _times(seed, P, K, t_bar):
    """Dwell times as an optimiser meets them: spread around the uniform start."""
    return t_bar * np.random.default_rng(seed).uniform(0.001, 2.0, size=(P, K))


def _stages(case):
    return [(s.split(":")[0], int(s.split(":")[1])) for s in case["stages"].split(",")]


def _batch_sizes(case):
    # the sizes belong to the case, the geometry to the seed
    r = np.random.default_rng(1000 + case["n"])
    return [(int(r.integers(case["K0"], case["K1"] + 1)), int(r.integers(case["M0"], case["M1"] + 1)))
            for _ in range(case["n"])]


def _rows(case, seed):
    """Training rows: plan inputs (weights, distance histograms) and smooth targets."""
    r = np.random.default_rng(seed)
    X = np.zeros((case["rows"], case["n_in"]), dtype=np.float32)
    X[:, :4] = _weights(seed + 1, case["rows"])
    h = np.abs(r.normal(size=(16, case["n_in"] - 4)))
    X[:, 4:] = (h / h.sum(1, keepdims=True))[r.integers(0, 16, case["rows"])]
    A = r.normal(size=(case["n_in"], case["n_out"])) * 0.5
    Y = np.abs(1.0 + np.tanh(X @ A)).astype(np.float32)
    sizes = [case["n_in"]] + [case["hidden"]] * case["depth"] + [case["n_out"]]
    p0 = np.concatenate([np.concatenate([r.uniform(-1, 1, size=o * i) * math.sqrt(6.0 / i), np.zeros(o)])
                         for i, o in zip(sizes[:-1], sizes[1:])]).astype(np.float32)
    need = case["steps"] * case["B"]
    order = np.concatenate([r.permutation(case["rows"]) for _ in range(-(-need // case["rows"]))])[:need]
    return sizes, X, Y, p0, order.astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        sizes, X, Y, p0, order = _rows(case, seed)
        net = Network(sizes, max_batch=case["B"])
        net.set_data(X, Y)
        return dict(kind=kind, net=net, p0=p0, order=order, B=case["B"])
    if kind == "batch":
        pls, Ws = [], []
        for i, (K, M) in enumerate(_batch_sizes(case)):
            kw = _geometry(seed * 64 + i, K, M)
            pl = Planner(dtype=case["dtype"], max_plans=case["P"])
            pl.load_case(**kw)
            pls.append(pl)
            Ws.append(_weights(seed * 64 + i + 32, case["P"]))
        return dict(kind=kind, planners=pls, W=Ws, stages=_stages(case), eps=case["eps"])
    K, M, P = case["K"], case["M"], case["P"]
    kw = _geometry(seed, K, M, case.get("Md"))
    W = _weights(seed + 1, P)
    if kind == "patient":
        t = _times(seed + 2, P, K, _start_time(kw, _dose_rate(kw["dwell_xyz"], kw["point_xyz"])))
        return dict(kind=kind, planner=Planner(dtype=case["dtype"], max_plans=P), kw=kw, W=W, x=np.sqrt(t))
    pl = Planner(dtype=case.get("dtype", "f32acc64"), max_plans=P)
    pl.load_case(**kw)
    if kind == "plan":
        return dict(kind=kind, planner=pl, W=W, stages=_stages(case), eps=case["eps"], finish=case["finish"])
    t = _times(seed + 2, P, K, _start_time(kw, _dose_rate(kw["dwell_xyz"], kw["point_xyz"])))
    if kind == "quality":
        pl.set_weights(W, t)
        return dict(kind=kind, planner=pl)
    pl.set_weights(W)
    x = np.sqrt(t)
    if case["arrays"] == "host":
        return dict(kind=kind, planner=pl, x=x)
    dev = dict(dtype=torch.float64, device=DEVICE)
    return dict(kind=kind, planner=pl, x=torch.tensor(x, **dev), F=torch.empty(P, **dev), g=torch.empty(P, K, **dev))


# ---- one pass ----

def _quality(pl):
    m = pl.metrics()
    best, cls, nd, frac = pl.select_plan()
    return dict(metrics=m, best=best, cls=cls, nondominated=nd, fraction=frac)


def run(state):
    kind = state["kind"]
    if kind == "train":
        net = state["net"]
        net.set_params(state["p0"])
        loss = net.train(state["order"], state["B"], 1e-3)
        return dict(loss=loss, params=net.params())
    if kind == "batch":
        for pl, W in zip(state["planners"], state["W"]):
            pl.set_weights(W)
        for k, (dt, cap) in enumerate(state["stages"]):
            optimize_many(state["planners"], max_iter=cap, eps=state["eps"], dtype=dt, resume_stopped=k > 0)
        return [pl.dwell_times() for pl in state["planners"]]
    pl = state["planner"]
    if kind == "evaluate":
        if "F" not in state:
            return pl.evaluate(state["x"])
        pl.evaluate_noalloc(state["x"].data_ptr(), state["F"].data_ptr(), state["g"].data_ptr())
        return state["F"], state["g"]
    if kind == "quality":
        return _quality(pl)
    if kind == "patient":
        pl.load_case(**state["kw"])
        pl.set_weights(state["W"])
        F, g = pl.evaluate(state["x"])
        return pl.start_time(), F, g
    pl.set_weights(state["W"])
    for k, (dt, cap) in enumerate(state["stages"]):
        pl.optimize(max_iter=cap, eps=state["eps"], dtype=dt, resume_stopped=k > 0)
    out = dict(t=pl.dwell_times())
    if state["finish"]:
        out["quality"] = _quality(pl)
    return out


# ---- what a pass cannot do without ----

def _evaluations(K, M, P, n, elem):
    """n evaluations of P plans: D and x read and g written once each, two products."""
    return n * (M * K * elem + 8.0 * P * K), n * 4.0 * M * K * P


def work(case):
    kind = case["kind"]
    elem = {"bf16": 2, "fp8": 1}
    if kind == "train":
        w = [case["n_in"]] + [case["hidden"]] * case["depth"] + [case["n_out"]]
        n = sum(i * o + o for i, o in zip(w[:-1], w[1:]))
        rows = case["B"] * (case["n_in"] + case["n_out"])
        # weights, moments and gradients read and written by Adam; the products' operands
        return dict(bytes=case["steps"] * 4.0 * (rows + 7 * n), flops=case["steps"] * 6.0 * case["B"] * n)
    if kind == "batch":
        parts = [_evaluations(K, M, case["P"], case["evaluations"], 4) for K, M in _batch_sizes(case)]
        return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))
    K, M, P = case["K"], case["M"], case["P"]
    if kind == "evaluate":
        e = elem.get(case["dtype"], 4)
        return dict(bytes=M * K * e + 16.0 * P * K, flops=4.0 * M * K * P)
    if kind == "plan":
        b, f = _evaluations(K, M, P, case["evaluations"], 4)
        if case["finish"]:  # the FP64 dose of the finished plans
            b, f = b + 8.0 * M * K, f + 2.0 * M * K * P
        return dict(bytes=b, flops=f)
    if kind == "quality":
        n = M + case["Md"]
        return dict(bytes=8.0 * n * K + 4.0 * P * K + 400.0 * P, flops=2.0 * n * K * P)
    e = elem.get(case["dtype"], 4)
    # the FP64 and the run-precision matrix written once, then one evaluation
    return dict(bytes=24.0 * M + M * K * (8.0 + e) + 16.0 * P * K, flops=12.0 * M * K + 4.0 * M * K * P)


# ---- the same in 64 bits, without the framework ----

def _params64(kw):
    g = torch.tensor(kw["group"].astype(np.int64), device=DEVICE)
    prm = torch.tensor(kw["group_params"], dtype=torch.float64, device=DEVICE)[g]
    organ = kw.get("group_organ", np.arange(8, dtype=np.int32))[kw["group"]].astype(np.int64)
    o = torch.tensor(organ, device=DEVICE)
    n = torch.bincount(o, minlength=4).double()
    return prm, o, n


def _evaluate64(kw, D, W, x):
    prm, o, n = _params64(kw)
    x = torch.tensor(x, dtype=torch.float64, device=DEVICE)
    w = (torch.tensor(W, dtype=torch.float64, device=DEVICE) / n)[:, o]
    d = (x * x) @ D.T
    lo, hi = (d - prm[:, 1]).clamp(max=0.0), (d - prm[:, 2]).clamp(min=0.0)
    kap = prm[:, 0] * lo + prm[:, 3] * hi
    F = (w * kap * (lo + hi)).sum(1)
    return F, 4.0 * x * ((w * kap) @ D)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        sizes, X, Y, p0, order = _rows(case, seed)
        X, Y, p = (torch.tensor(v, dtype=torch.float64, device=DEVICE) for v in (X, Y, p0))
        m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
        for s in range(case["steps"]):
            i = torch.tensor(order[s * case["B"]:(s + 1) * case["B"]].astype(np.int64), device=DEVICE)
            q = p.clone().requires_grad_(True)
            h, off = X[i], 0
            for k, (a, b) in enumerate(zip(sizes[:-1], sizes[1:])):
                h = h @ q[off:off + a * b].view(b, a).T + q[off + a * b:off + a * b + b]
                off += a * b + b
                h = h.relu() if k < len(sizes) - 2 else h
            loss = ((h - Y[i]) ** 2).mean()
            g, = torch.autograd.grad(loss, q)
            losses.append(float(loss))
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            p = p - 1e-3 * (m / (1 - 0.9 ** (s + 1))) / ((v / (1 - 0.999 ** (s + 1))).sqrt() + 1e-8)
        return dict(loss=sum(losses) / len(losses), params=p)
    if kind in ("plan", "batch"):
        # no such value: the line searches' accept decisions follow the run's rounding
        return None
    kw = _geometry(seed, case["K"], case["M"], case.get("Md"))
    W = _weights(seed + 1, case["P"])
    D = _dose_rate(kw["dwell_xyz"], kw["point_xyz"])
    t_bar = _start_time(kw, D)
    t = _times(seed + 2, case["P"], case["K"], t_bar)
    if kind == "evaluate":
        return _evaluate64(kw, D, W, np.sqrt(t))
    if kind == "patient":
        return (t_bar,) + tuple(_evaluate64(kw, D, W, np.sqrt(t)))
    # quality: the planner holds x = sqrt(t) in FP32
    x = torch.tensor(np.sqrt(t).astype(np.float32), device=DEVICE).double()
    tt = x * x
    prm, o, n = _params64(kw)
    d = tt @ D.T
    lo, hi = (d - prm[:, 1]).clamp(max=0.0), (d - prm[:, 2]).clamp(min=0.0)
    f = prm[:, 0] * lo * lo + prm[:, 3] * hi * hi
    fo = torch.stack([f[:, o == j].sum(1) / n[j] for j in range(4)], 1)
    if "dvh_xyz" in kw:
        d = tt @ _dose_rate(kw["dwell_xyz"], kw["dvh_xyz"]).T
        o = torch.tensor(kw["dvh_organ"].astype(np.int64), device=DEVICE)
    vol = torch.tensor(kw["volume_cc"], dtype=torch.float64, device=DEVICE)
    cols = dict(V100_pct=[], V75_cc=[], D10_pct=[], D90_pct=[])
    for j in range(4):
        dj = d[:, o == j]
        nj = dj.shape[1]
        cols["V100_pct"].append(100.0 * (dj >= RX).double().mean(1))
        cols["V75_cc"].append(vol[j] * (dj >= 0.75 * RX).double().mean(1))
        for name, pct in (("D10_pct", 10), ("D90_pct", 90)):
            k = max(1, -(-pct * nj // 100))
            cols[name].append(100.0 / RX * torch.kthvalue(dj, nj - k + 1, dim=1).values)
    m = {name: torch.stack(c, 1) for name, c in cols.items()}
    m.update(F64=(torch.tensor(W, dtype=torch.float64, device=DEVICE) * fo).sum(1), f_organ=fo, F_run=None,
             iterations=None, evaluations=None, status=None)
    return dict(metrics=m, best=None, cls=None, nondominated=None, fraction=None)
