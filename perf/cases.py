"""The planner's performance cases: what each stands for in use, its inputs,
one pass through the public entry points, the work a pass cannot do without,
and its outputs in 64 bits.

Sizes are those of the repository's workloads: a 10 km box with 50 to 100
known plans and 81 actions; 2000 plans over a terrain heightmap with 81
actions; 3000 plans with 360 actions at half-second steps.  `draw` spreads
over the same ranges.  A planning case returns whole trajectories (points,
actions, values, outcomes); a planner's table is rewound, as part of the
pass, where planning has added to it.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2008_03518_amd import fastmdp as fm
from paper_2008_03518_amd import proposal
from paper_2008_03518_amd import scenario as S

CLIMBS = {1: (0.0,), 3: (-5.0, 0.0, 5.0), 5: (-5.0, -2.5, 0.0, 2.5, 5.0)}
SPEEDS = {1: (30.0,), 2: (20.0, 40.0), 3: (20.0, 30.0, 40.0)}
SMALL = dict(box_km=10, dt=1.0, heads=9, climbs=3, speeds=3, terrain=False, range_query=False, window=1)
PAPER = dict(box_km=30, dt=1.0, heads=9, climbs=3, speeds=3, terrain=True, range_query=False, window=1)
LARGE = dict(box_km=30, dt=0.5, heads=24, climbs=5, speeds=3, terrain=False, range_query=False, window=1)
RANGE = dict(LARGE, range_query=True)
LR = 1e-5            # a late training step's rate (decayed from the start's 2e-3)
TRAIN_STEPS = 8      # training steps per pass
ROW_STEP = 7         # rows between two departure candidates


def listed():
    return [
        # one state scored, every term of every action returned: the smallest call
        dict(SMALL, name="step", kind="step", plans=50),
        # the paper's mode of operation at small scale: plan a request, commit it, plan the next
        dict(SMALL, name="sequential_small", kind="sequential", plans=50, requests=5),
        # one request of an operator against a full airspace, range query on
        dict(RANGE, name="request_range", kind="request", plans=3000),
        # the same request from several departure rows (ground delay)
        dict(RANGE, name="departures", kind="departures", plans=3000, requests=13),
        # aircraft planned together, each aware of the others
        dict(SMALL, name="batch", kind="batch", plans=100, requests=10),
        # the headline: a stream of requests against 3000 plans, range query on
        dict(RANGE, name="fcfs_range", kind="fcfs", plans=3000, requests=1000, propose="none"),
        # the same method with every plan swept at every step
        dict(LARGE, name="fcfs_full", kind="fcfs", plans=3000, requests=1000, propose="none"),
        # a request stream over terrain at the paper's scale
        dict(PAPER, name="fcfs_terrain", kind="fcfs", plans=2000, requests=200, propose="none"),
        # the action proposal with its exact certificate (goal ranking, top 8)
        dict(LARGE, name="fcfs_goal", kind="fcfs", plans=3000, requests=300, propose="goal"),
        # the paper's ten-step scoring window
        dict(RANGE, name="fcfs_window", kind="fcfs", plans=3000, requests=100, propose="none", window=10),
        # training data of the proposal: traffic features of many states
        dict(LARGE, name="features", kind="features", plans=3000, states=100000),
        # training the proposal network: steps on batches that are on the GPU
        dict(name="train", kind="train", batch=4096, outputs=360),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "sequential", "request", "departures", "batch", "fcfs", "fcfs", "fcfs", "features",
                       "train"])
    if kind == "train":
        return dict(kind=kind, batch=32 * _log_int(rng, 1, 128), outputs=rng.choice([81, 240, 360, 510]))
    # action sets from 27 (9 x 3 x 1) to 510 (34 x 5 x 3)
    heads, climbs, speeds = rng.choice([(9, 3, 1), (9, 3, 3), (13, 3, 2), (16, 5, 3), (24, 5, 3), (34, 5, 3)])
    small = kind == "batch" or rng.random() < 0.3
    case = dict(kind=kind, box_km=10 if small else 30, dt=rng.choice([0.5, 1.0]), heads=heads, climbs=climbs,
                speeds=speeds, terrain=not small and rng.random() < 0.25, range_query=rng.random() < 0.6, window=1,
                plans=_log_int(rng, 30, 150) if small else _log_int(rng, 500, 3400))
    if kind == "sequential":
        case["requests"] = rng.randint(2, 6)
    elif kind == "departures":
        case["requests"] = rng.randint(2, 40)
    elif kind == "batch":
        case["requests"] = rng.randint(2, 20)
        case["range_query"] = False
    elif kind == "features":
        case["states"] = _log_int(rng, 100, 100000)
        case["range_query"] = False
    elif kind == "fcfs":
        case["requests"] = _log_int(rng, 5, 40) if small else _log_int(rng, 20, 500)
        case["propose"] = rng.choice(["none", "none", "goal"])
        if case["propose"] == "none" and rng.random() < 0.2:
            case["window"] = rng.choice([2, 5])
            case["requests"] = min(case["requests"], 100)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _config(case):
    L = 1000.0 * case["box_km"]
    rows = 3601
    cap = (case["plans"] + case.get("requests", 1) + 64 + 3) // 4 * 4
    return S.Config(box_min=(0.0, 0.0, 0.0), box_max=(L, L, 1000.0 if case["box_km"] == 10 else 1500.0), dt=case["dt"],
                    n_head=case["heads"], climb=CLIMBS[case["climbs"]], speed=SPEEDS[case["speeds"]],
                    max_steps=3600, plan_capacity=max(cap, 256), max_rows=rows + 16, lookahead=case["window"],
                    range_query=1 if case["range_query"] else 0)


def _scenario(case, seed):
    """Known plans, requests and terrain of the repository's recipe."""
    cfg = _config(case)
    rng = np.random.default_rng(seed)
    terrain = S.make_terrain(rng, cfg) if case["terrain"] else None
    plans = S.make_known_plans(rng, cfg, case["plans"], terrain)
    n_req = {"fcfs": case.get("requests", 1), "sequential": case.get("requests", 1),
             "batch": case.get("requests", 1), "features": 200}.get(case["kind"], 1)
    req = S.make_requests(rng, cfg, n_req, plans, terrain)
    return S.Scenario(case["kind"], cfg, plans, req, terrain, seed)


def _departure_rows(case):
    return np.arange(case["requests"], dtype=np.int32) * ROW_STEP


def _flight_states(sc, n, seed):
    """States along the requests' straight tracks, in flight order: positions,
    goals and rows."""
    rng = np.random.default_rng(seed)
    r, step = sc.requests, max(sc.cfg.speed) * sc.cfg.dt
    dist = np.linalg.norm(r.goal - r.origin, axis=1)
    count = np.maximum((dist / step).astype(np.int64), 1)
    which = rng.choice(r.n, size=n, p=count / count.sum())
    k = (rng.random(n) * count[which]).astype(np.int64)
    order = np.lexsort((k, which))
    which, k = which[order], k[order]
    f = (k / count[which])[:, None]
    pos = r.origin[which] + f * (r.goal[which] - r.origin[which])
    return pos, r.goal[which].copy(), np.minimum(k, sc.cfg.max_rows - 2).astype(np.int32)


def _train_inputs(case, seed):
    """A trained-size network's parameters and batches shaped like the
    proposal's features (sparse closeness and count features, dense geometry)."""
    rng = np.random.default_rng(seed)
    params = proposal.init_params(case["outputs"], seed)
    for b in ("b1", "b2", "b3"):
        params[b] = rng.uniform(-0.05, 0.05, params[b].shape)
    n = TRAIN_STEPS * case["batch"]
    x = np.zeros((n, fm.N_FEAT), dtype=np.float32)
    near = rng.random((n, 32)) < 0.05
    x[:, :32] = np.where(near, rng.random((n, 32)), 0.0)
    x[:, 32:64] = np.where(near, rng.integers(1, 5, (n, 32)) / 4.0, 0.0)
    x[:, 64:76] = rng.uniform(-1.0, 1.0, (n, 12))
    y = np.minimum(rng.geometric(0.1, n) - 1, case["outputs"] - 1).astype(np.int32)
    return params, x, y


def _plan_rows(m, capacity):
    """m plans whose buffers are rows of three arrays, which a program can
    hand on whole; entries past a plan's points stay zero."""
    xyz, action, value = np.zeros((m, capacity, 3)), np.zeros((m, capacity), np.int32), np.zeros((m, capacity))
    plans = []
    for i in range(m):
        p = fm.Plan(0)
        p.xyz, p.action, p.value = xyz[i], action[i], value[i]
        p.c.capacity = capacity
        p.c.xyz = xyz[i].ctypes.data_as(ctypes.POINTER(ctypes.c_double))
        p.c.action = action[i].ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
        p.c.value = value[i].ctypes.data_as(ctypes.POINTER(ctypes.c_double))
        plans.append(p)
    return plans, dict(xyz=xyz, action=action, value=value)


def prepare(case, seed):
    st = dict(kind=case["kind"], case=case)
    if case["kind"] == "train":
        params, x, y = _train_inputs(case, seed)
        net = fm.Mlp(case["outputs"], max_batch=case["batch"])
        net.set_params(params)
        st.update(net=net, x=fm.DeviceArray.from_host(x), y=fm.DeviceArray.from_host(y))
        return st
    sc = _scenario(case, seed)
    kind, m = case["kind"], case.get("requests", 1)
    ctx = fm.context_for(sc, max_slots={"fcfs": 1024, "batch": 32}.get(kind, m))
    st.update(ctx=ctx, req=sc.requests)
    if kind in ("sequential", "fcfs"):
        ctx.snapshot()
    if kind not in ("step", "features"):
        st["plans"], st["arrays"] = _plan_rows(m, ctx.capacity)
    if kind == "step":
        # a third of the way along the straight track
        o, g = sc.requests.origin[0], sc.requests.goal[0]
        d = np.linalg.norm(g - o)
        k = int(d / (max(sc.cfg.speed) * sc.cfg.dt) / 3.0)
        st.update(pos=o + (g - o) / 3.0, goal=g, row=k)
    elif kind == "departures":
        st["rows"] = _departure_rows(case)
    elif kind == "fcfs":
        if case["propose"] == "goal":
            ctx.set_proposal(fm.PROPOSE_GOAL, 8, refresh=64)
    elif kind == "features":
        pos, goal, rows = _flight_states(sc, case["states"], seed)
        seqs = np.full(case["states"], ctx.next_seq(), dtype=np.int32)
        st.update(pos=fm.DeviceArray.from_host(pos), goal=fm.DeviceArray.from_host(goal),
                  rows=fm.DeviceArray.from_host(rows), seqs=fm.DeviceArray.from_host(seqs))
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

class _OnDevice:
    """The library's device array as torch reads it (no copy)."""

    def __init__(self, a):
        self.a = a
        self.__cuda_array_interface__ = dict(shape=a.shape, typestr=a.dtype.str, data=(a.ptr, False), version=3,
                                             strides=None)


def _whole(state, plans):
    """The plans' points, actions, values, lengths and outcomes in the state's
    arrays (entries past a plan's points stay zero)."""
    a = state["arrays"]
    for i, p in enumerate(plans):
        n = p.n_points
        a["xyz"][i, :n], a["action"][i, :n], a["value"][i, :n] = p.points(), p.actions(), p.values()
    return _outcomes(a, plans)


def _outcomes(arrays, plans):
    return dict(arrays, status=np.array([p.status for p in plans], dtype=np.int32),
                n_points=np.array([p.n_points for p in plans], dtype=np.int32))


def run(state):
    kind, ctx = state["kind"], state.get("ctx")
    if kind == "step":
        return ctx.eval_step(state["pos"], state["goal"], state["row"])
    if kind == "request":
        r = state["req"]
        return _whole(state, [ctx.plan_request(r.origin[0], r.goal[0], int(r.t0[0]))])
    if kind == "sequential":
        r = state["req"]
        ctx.rewind()
        out, committed = [], []
        for i in range(r.n):
            p = ctx.plan_request(r.origin[i], r.goal[i], int(r.t0[i]))
            committed.append(p.status == fm.OK and ctx.commit_plan(p))
            out.append(p)
        return dict(_whole(state, out), committed=np.array(committed))
    if kind == "departures":
        r = state["req"]
        plans, chosen = ctx.plan_departures(r.origin[0], r.goal[0], state["rows"])
        return dict(_whole(state, plans), chosen=chosen)
    if kind == "batch":
        return _whole(state, ctx.plan_batch(state["req"]))
    if kind == "fcfs":
        ctx.rewind()
        plans, committed, _ = ctx.plan_fcfs(state["req"], out=state["plans"])
        return dict(_outcomes(state["arrays"], plans), committed=committed)
    if kind == "features":
        f = ctx.features(state["pos"], state["goal"], state["rows"], state["seqs"])
        return torch.as_tensor(_OnDevice(f), device="cuda")
    # train: steps on consecutive batches, then the weights
    net, b = state["net"], state["case"]["batch"]
    loss = [net.train_step(state["x"].rows(i * b, b), state["y"].rows(i * b, b), LR) for i in range(TRAIN_STEPS)]
    p = net.get_params()
    return dict({k: v.astype(np.float32) for k, v in p.items()}, loss=np.array(loss, dtype=np.float32))


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------

def work(case):
    if case["kind"] == "train":
        h, no, b = fm.MLP_HIDDEN, case["outputs"], case["batch"]
        macs = fm.N_FEAT * h + h * h + h * no
        n_par = macs + 2 * h + no
        # forward, and backward to weights and activations (none to the inputs)
        flops = 2.0 * b * (2 * macs + (macs - fm.N_FEAT * h))
        return {"bytes": float(TRAIN_STEPS * (b * (4 * fm.N_FEAT + 4) + 4 * 7 * n_par)),
                "flops": float(TRAIN_STEPS * flops)}
    L, A = 1000.0 * case["box_km"], case["heads"] * case["climbs"] * case["speeds"]
    ell = max(SPEEDS[case["speeds"]]) * case["dt"]
    mean = 0.5214 * L                       # mean distance of two points of a square
    P = case["plans"]
    steps = mean / ell                      # a flight's steps
    rows = mean / (30.0 * case["dt"])       # a known plan's rows
    active = P * min(1.0, rows / (rows + steps) + 0.3)     # plans of a row, over a flight
    if case["kind"] == "step":
        return {"bytes": 16.0 * P + 32.0 * A, "flops": 8.0 * A * P}
    if case["kind"] == "features":
        n = case["states"]
        return {"bytes": 16.0 * P * rows + n * (56.0 + 4 * fm.N_FEAT), "flops": 8.0 * n * active}
    n = case.get("requests", 1)
    table = 16.0 * P * min(rows, steps)     # the rows flown through, read once
    points = n * steps * 36.0
    if case["range_query"]:
        # a distance test per plan and step, then the value of every action
        flops = n * steps * (active * 4.0 + A * 40.0 * case["window"])
    else:
        flops = n * steps * active * A * 8.0 * case["window"]
    return {"bytes": table + points, "flops": flops}


# ---------------------------------------------------------------------------
# outputs in 64 bits
# ---------------------------------------------------------------------------

class _Table:
    """Known plans by row, FP32 as stored, held in FP64."""

    def __init__(self, cfg, plans):
        rows = [[] for _ in range(cfg.max_rows)]
        off = 0
        for t0, n in zip(plans.t0, plans.length):
            for k in range(int(n)):
                rows[int(t0) + k].append(off + k)
            off += int(n)
        pts = plans.xyz.astype(np.float64)
        self.rows = [pts[np.array(r, dtype=np.int64)] if r else np.zeros((0, 3)) for r in rows]

    def append(self, t0, xyz):
        stored = xyz.astype(np.float32).astype(np.float64)
        for k in range(xyz.shape[0]):
            self.rows[t0 + k] = np.concatenate([self.rows[t0 + k], stored[k: k + 1]])

    def row(self, t):
        return self.rows[t] if 0 <= t < len(self.rows) else np.zeros((0, 3))


def _height(ter, x, y):
    fx = np.clip((x - ter.x0) / ter.cell, 0.0, ter.nx - 1.0)
    fy = np.clip((y - ter.y0) / ter.cell, 0.0, ter.ny - 1.0)
    i, j = np.minimum(fx.astype(int), ter.nx - 2), np.minimum(fy.astype(int), ter.ny - 2)
    ax, ay = fx - i, fy - j
    h = ter.h.astype(np.float64)
    return (1 - ay) * ((1 - ax) * h[j, i] + ax * h[j, i + 1]) + ay * ((1 - ax) * h[j + 1, i] + ax * h[j + 1, i + 1])


def _score(cfg, table, terrain, s, g, t):
    """Every action's successor, terms and value at state s, row t."""
    b = g - s
    r = math.hypot(b[0], b[1])
    cb, sb = (b[0] / r, b[1] / r) if r > 0 else (1.0, 0.0)
    th = 2.0 * np.pi * np.arange(cfg.n_head) / cfg.n_head
    hx, hy = cb * np.cos(th) - sb * np.sin(th), sb * np.cos(th) + cb * np.sin(th)
    step, dz = np.array(cfg.speed) * cfg.dt, np.array(cfg.climb) * cfg.dt
    H, C, V = cfg.n_head, len(dz), len(step)
    p = np.empty((H, C, V, 3))
    p[..., 0] = s[0] + hx[:, None, None] * step[None, None, :]
    p[..., 1] = s[1] + hy[:, None, None] * step[None, None, :]
    p[..., 2] = s[2] + dz[None, :, None]
    p = p.reshape(-1, 3)
    G = cfg.r_goal * cfg.gamma ** (np.sqrt(((g - p) ** 2).sum(1)) / cfg.ell)
    I, T, clear = np.zeros(len(p)), np.zeros(len(p)), np.full(len(p), np.inf)
    q = table.row(t + 1)
    if len(q):
        reach = cfg.R_intr + math.hypot(max(step), max(abs(dz))) + 1.0
        q = q[((q - s) ** 2).sum(1) < reach * reach]
        if len(q):
            d = np.sqrt(((p[:, None, :] - q[None, :, :]) ** 2).sum(2)).min(1)
            I = np.where(d < cfg.R_intr, cfg.r_intr * cfg.gamma_intr ** (d / cfg.ell), 0.0)
    if terrain is not None:
        clear = p[:, 2] - _height(terrain, p[:, 0], p[:, 1])
        T = np.where(clear < cfg.R_terr, cfg.r_terr * cfg.gamma_terr ** (np.maximum(clear, 0.0) / cfg.ell), 0.0)
    out = ((p < np.array(cfg.box_min)) | (p > np.array(cfg.box_max))).any(1)
    Vv = np.where(out, -np.inf, G - np.maximum(I, T))
    vm = Vv.max()
    best = int(np.argmax(Vv >= vm - fm.TIE_REL * abs(vm))) if vm > -np.inf else -1
    return p, G, I, T, clear, Vv, best


def _fly(cfg, table, terrain, o, g, t0):
    xyz, act, val, s, status = [o.copy()], [-1], [0.0], o.copy(), None
    near = table.row(t0)
    if ((o < np.array(cfg.box_min)) | (o > np.array(cfg.box_max))).any() or \
            (len(near) and ((near - o) ** 2).sum(1).min() < cfg.R_sep ** 2) or \
            (terrain is not None and o[2] < _height(terrain, o[0], o[1])):
        status = fm.REJECT_ORIGIN
    while status is None:
        k = len(act) - 1
        if np.sqrt(((g - s) ** 2).sum()) <= cfg.ell:
            status = fm.OK
        elif k >= cfg.max_steps:
            status = fm.TIMEOUT
        else:
            p, _, I, _, clear, V, best = _score(cfg, table, terrain, s, g, t0 + k)
            if best < 0:
                status = fm.NO_VALID_ACTION
                break
            s = p[best]
            xyz.append(s)
            act.append(best)
            val.append(V[best])
            if I[best] > 0.0:
                status = fm.REJECT_SEPARATION
            elif clear[best] < 0.0:
                status = fm.REJECT_TERRAIN
    return status, np.array(xyz), np.array(act, dtype=np.int32), np.array(val)


def _valid(cfg, table, terrain, t0, xyz):
    for k, x in enumerate(xyz):
        q = table.row(t0 + k)
        if len(q) and ((q - x) ** 2).sum(1).min() < cfg.R_sep ** 2:
            return False
    return terrain is None or bool((xyz[:, 2] >= _height(terrain, xyz[:, 0], xyz[:, 1])).all())


def _whole_exact(cfg, flights):
    _, a = _plan_rows(len(flights), cfg.max_steps + 1)
    for i, (_, xyz, act, val) in enumerate(flights):
        n = len(act)
        a["xyz"][i, :n], a["action"][i, :n], a["value"][i, :n] = xyz, act, val
    return dict(a, status=np.array([f[0] for f in flights], dtype=np.int32),
                n_points=np.array([len(f[1]) for f in flights], dtype=np.int32))


def _exact_features(case, seed):
    sc = _scenario(case, seed)
    pos, goal, rows = _flight_states(sc, case["states"], seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    n_rows, cap = sc.cfg.max_rows, case["plans"]
    tab = np.full((n_rows, cap, 3), np.nan, dtype=np.float32)     # column = plan index
    off = sc.plans.offsets()
    for j in range(sc.plans.n):
        t0, n = int(sc.plans.t0[j]), int(sc.plans.length[j])
        tab[t0: t0 + n, j] = sc.plans.xyz[off[j]: off[j + 1]]
    tab = torch.from_numpy(tab).to(dev)
    lo = torch.tensor(sc.cfg.box_min, dtype=torch.float64, device=dev)
    hi = torch.tensor(sc.cfg.box_max, dtype=torch.float64, device=dev)
    R, out = 600.0, []
    for i in range(0, len(pos), 1024):
        s = torch.from_numpy(pos[i: i + 1024]).to(dev)
        g = torch.from_numpy(goal[i: i + 1024]).to(dev)
        r = torch.from_numpy(rows[i: i + 1024].astype(np.int64) + 1).to(dev)
        q = tab[r].double() - s[:, None, :]
        d = q.square().sum(2).sqrt()
        close = d < R                                             # NaN: no entry
        b = g - s
        rh = b[:, :2].square().sum(1).sqrt()
        u = torch.where(rh[:, None] > 0, b[:, :2] / rh[:, None], torch.tensor([1.0, 0.0], dtype=torch.float64, device=dev))
        along = q[..., 0] * u[:, None, 0] + q[..., 1] * u[:, None, 1]
        cross = q[..., 1] * u[:, None, 0] - q[..., 0] * u[:, None, 1]
        sec = torch.floor((torch.atan2(cross, along) + math.pi) * 16.0 / (2.0 * math.pi)).clamp(0, 15)
        idx = torch.where(close, 2 * sec + (q[..., 2] < 0), torch.full_like(sec, 32.0)).long()
        near = torch.zeros(len(s), 33, dtype=torch.float64, device=dev)
        near.scatter_reduce_(1, idx, torch.where(close, 1.0 - d / R, torch.zeros_like(d)), "amax")
        cnt = torch.zeros(len(s), 33, dtype=torch.float64, device=dev)
        cnt.scatter_add_(1, idx, close.double())
        n = close.sum(1)
        d3 = b.square().sum(1).sqrt()
        f = torch.zeros(len(s), fm.N_FEAT, dtype=torch.float64, device=dev)
        f[:, :32] = near[:, :32]
        f[:, 32:64] = cnt[:, :32].clamp(max=4) / 4.0
        f[:, 64], f[:, 65] = rh / 10000.0, b[:, 2] / 500.0
        f[:, 66], f[:, 67] = d3 / sc.cfg.ell / 1000.0, torch.log1p(d3 / sc.cfg.ell) / 8.0
        f[:, 68] = s[:, 2] / 1000.0
        f[:, 69] = (s[:, 2] - lo[2]) / (hi[2] - lo[2])
        f[:, 70:72] = (s[:, :2] - lo[:2]) / (hi[:2] - lo[:2])
        f[:, 72:74] = u
        f[:, 74] = (n / 16.0).clamp(max=1.0)
        f[:, 75] = torch.where(close, d, torch.full_like(d, R)).min(1).values / R
        out.append(f)
    return torch.cat(out)


def _exact_train(case, seed):
    params, x, y = _train_inputs(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    names = ("W1", "b1", "W2", "b2", "W3", "b3")
    p = {k: torch.tensor(params[k].astype(np.float32), dtype=torch.float64, device=dev) for k in names}
    m = {k: torch.zeros_like(v) for k, v in p.items()}
    v2 = {k: torch.zeros_like(v) for k, v in p.items()}
    X, Y, b, loss = torch.from_numpy(x).to(dev).double(), torch.from_numpy(y).to(dev).long(), case["batch"], []
    for t in range(1, TRAIN_STEPS + 1):
        xb, yb = X[(t - 1) * b: t * b], Y[(t - 1) * b: t * b]
        h1 = (xb @ p["W1"] + p["b1"]).clamp(min=0)
        h2 = (h1 @ p["W2"] + p["b2"]).clamp(min=0)
        z = h2 @ p["W3"] + p["b3"]
        loss.append(float((torch.logsumexp(z, 1) - z[torch.arange(b, device=dev), yb]).mean()))
        d3 = torch.softmax(z, 1)
        d3[torch.arange(b, device=dev), yb] -= 1.0
        d3 /= b
        d2 = (d3 @ p["W3"].T) * (h2 > 0)
        d1 = (d2 @ p["W2"].T) * (h1 > 0)
        grad = dict(W3=h2.T @ d3, b3=d3.sum(0), W2=h1.T @ d2, b2=d2.sum(0), W1=xb.T @ d1, b1=d1.sum(0))
        for k in names:
            m[k] = 0.9 * m[k] + 0.1 * grad[k]
            v2[k] = 0.999 * v2[k] + 0.001 * grad[k] ** 2
            p[k] = p[k] - LR * (m[k] / (1 - 0.9 ** t)) / ((v2[k] / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return dict({k: v.cpu().numpy() for k, v in p.items()}, loss=np.array(loss))


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "features":
        return _exact_features(case, seed)
    if kind in ("batch", "fcfs"):
        return None
    sc = _scenario(case, seed)
    cfg, table, ter = sc.cfg, _Table(sc.cfg, sc.plans), sc.terrain
    r = sc.requests
    o, g = r.origin[0], r.goal[0]
    if kind == "step":
        d = np.linalg.norm(g - o)
        k = int(d / (max(cfg.speed) * cfg.dt) / 3.0)
        _, G, I, T, _, V, best = _score(cfg, table, ter, o + (g - o) / 3.0, g, k)
        return dict(V=V, G=G, I=I, T=T, best=best)
    if kind == "request":
        return _whole_exact(cfg, [_fly(cfg, table, ter, o, g, int(r.t0[0]))])
    if kind == "departures":
        rows = _departure_rows(case)
        fl = [_fly(cfg, table, ter, o, g, int(t)) for t in rows]
        ok = [i for i, f in enumerate(fl) if f[0] == fm.OK and _valid(cfg, table, ter, int(rows[i]), f[1])]
        return dict(_whole_exact(cfg, fl), chosen=ok[0] if ok else -1)
    fl, committed = [], []
    for i in range(r.n):
        f = _fly(cfg, table, ter, r.origin[i], r.goal[i], int(r.t0[i]))
        c = f[0] == fm.OK and _valid(cfg, table, ter, int(r.t0[i]), f[1])
        if c:
            table.append(int(r.t0[i]), f[1])
        fl.append(f)
        committed.append(c)
    return dict(_whole_exact(cfg, fl), committed=np.array(committed))
