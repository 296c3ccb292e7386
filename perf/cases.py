"""The performance cases of this framework: the calls its users make, over the
sizes they make them at, each through a public entry point.

Kinds of work (field "kind"):

    search     Searcher.search: one frame from host memory to the best pass on
               the host, with its feasibility and score maps on the device
    resident   Batch.run(graph=True): a device-resident batch of frames with
               windows of uneven size, replayed at its tuned launch shape
    requests   Searcher.search_batch: several frames staged from host memory
               (a serving loop's batch), best passes and maps on the device
    sweep      Searcher.ray_search: kick directions x powers
    power      Searcher.search_power: every point at its own kick speed
    shot       Searcher.shot: shooting decisions, from the ball or as a map
    running    Searcher.running_points: best running point of every zone
    forward    Mlp.forward: the network's predicted maps
    train      Mlp.train_step: consecutive training steps, then the weights
    proposals  Mlp.search on a resident batch: network, top cells re-scored
               exactly, exact fallback
    proposals_host  Mlp.search_frames: the same from host memory to the host

Frames are drawn from the seed by the framework's own generator (positions
uniform on the field, velocities uniform in a 1.5 m/s disc).  `exact` gives the
float64 value of each computed map in plain torch.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_1909_07717_amd
from paper_1909_07717_amd import binding as B
from paper_1909_07717_amd import flops as FL
from paper_1909_07717_amd import framegen as G
from paper_1909_07717_amd.zones import front_zones

WEIGHTS = os.path.join(os.path.dirname(paper_1909_07717_amd.__file__), "weights", "surrogate.npz")
CELLS = 2806
SPACINGS = (0.05, 0.1, 0.2)


def listed():
    return [
        # one frame per decision at the coarsest grid: 6v6, one flat speed
        dict(name="frame_small", kind="search", n_team=6, n_opp=6, h=0.2, speeds=1, chip=False,
             K=64, reduced=False),
        # the headline frame: 8v8, 5 cm, 16 speeds flat and chip
        dict(name="frame_full", kind="search", n_team=8, n_opp=8, h=0.05, speeds=16, chip=True,
             K=256, reduced=False),
        # offline analysis of many game states: uneven windows, 8 flat speeds
        dict(name="batch_windows", kind="resident", n=256, speeds=8, chip=False, K=128,
             reduced=False),
        # one admitted batch of the serving loop: mixed 20/10/5 cm grids, 4-16 speeds
        dict(name="serving_requests", kind="requests", n=16, K=128, reduced=True),
        # the paper's own form: 128 directions x 64 powers
        dict(name="sweep_paper", kind="sweep", n=512, n_team=8, n_opp=8, dirs=128, speeds=64,
             chip=False, K=256),
        # the kick speed of every point of the field
        dict(name="power_full", kind="power", n=1, n_team=8, n_opp=8, h=0.05, K=256),
        # where on the field a shot succeeds
        dict(name="shot_map", kind="shot", n=1, n_team=8, n_opp=8, h=0.05, K=256, map=True),
        # four front zones that follow the ball, for many frames
        dict(name="running_zones", kind="running", n=2048, n_team=8, n_opp=8),
        # predicted maps of a batch
        dict(name="network_forward", kind="forward", n=4096, n_team=6, n_opp=6),
        # a stretch of training between two checkpoints
        dict(name="network_train", kind="train", n=4000, steps=64, n_team=6, n_opp=6),
        # one frame per decision through the network
        dict(name="proposals_one", kind="proposals_host", n=1, k=64, n_team=6, n_opp=6),
        # a batch through the network
        dict(name="proposals_batch", kind="proposals", n=1000, k=64, n_team=6, n_opp=6),
    ]


def draw(rng):
    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["search", "search", "resident", "requests", "sweep", "power", "shot",
                       "running", "forward", "train", "proposals", "proposals_host"])
    team, opp = rng.randint(3, 11), rng.randint(2, 11)
    K = rng.choice([64, 128, 192, 256])
    if kind == "search":
        return dict(kind=kind, n_team=team, n_opp=opp, h=rng.choice(SPACINGS),
                    speeds=rng.randint(1, 16), chip=rng.random() < 0.5, K=K,
                    reduced=rng.random() < 0.3)
    if kind == "resident":
        return dict(kind=kind, n=between(2, 250), speeds=rng.randint(4, 8), chip=False,
                    K=rng.choice([64, 128]), reduced=rng.random() < 0.5)
    if kind == "requests":
        return dict(kind=kind, n=between(1, 15), K=rng.choice([64, 128]),
                    reduced=rng.random() < 0.5)
    if kind == "sweep":
        return dict(kind=kind, n=between(1, 500), n_team=rng.randint(3, 8),
                    n_opp=rng.randint(2, 8), dirs=rng.choice([32, 90, 128]),
                    speeds=rng.randint(8, 32), chip=rng.random() < 0.5, K=K)
    if kind == "power":
        return dict(kind=kind, n=1, n_team=team, n_opp=opp, h=rng.choice(SPACINGS), K=K)
    if kind == "shot":
        if rng.random() < 0.5:
            return dict(kind=kind, n=between(1, 4096), n_team=team, n_opp=opp, h=0.2, K=K,
                        map=False)
        return dict(kind=kind, n=1, n_team=team, n_opp=opp, h=rng.choice(SPACINGS), K=K, map=True)
    if kind == "running":
        return dict(kind=kind, n=between(1, 2000), n_team=team, n_opp=opp)
    if kind == "forward":
        return dict(kind=kind, n=between(1, 4096), n_team=rng.randint(3, 8),
                    n_opp=rng.randint(2, 8))
    if kind == "train":
        return dict(kind=kind, n=between(250, 4000), steps=rng.randint(16, 64), n_team=6, n_opp=6)
    if kind == "proposals":
        return dict(kind=kind, n=between(16, 1000), k=rng.choice([16, 64]), n_team=6, n_opp=6)
    return dict(kind=kind, n=between(1, 64), k=rng.choice([16, 64]), n_team=6, n_opp=6)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _speeds(case):
    return [4.0] if case["speeds"] == 1 else G.speeds_linear(case["speeds"])


def _frames(case, seed):
    """The case's frames (framegen frames with windows and variants): robot
    states from the seed; counts, windows, speeds and, for the zones that
    follow it, the ball's x from the case, so that a case has one size."""
    rng, shape = np.random.default_rng(seed), np.random.default_rng(case.get("n", 1))
    kind = case["kind"]
    out = []
    for _ in range(case.get("n", 1)):
        if kind in ("resident", "requests"):
            f = G.random_frame(rng, int(shape.integers(6, 9)), int(shape.integers(6, 9)))
        else:
            f = G.random_frame(rng, case["n_team"], case["n_opp"])
        f.windows = [G.full_window(case.get("h", 0.2))]
        f.variants = [(G.FLAT, 4.0)]
        if kind == "resident":
            f.windows = [G.random_window(shape)]
        elif kind == "requests":
            f.windows = [G.full_window(float(shape.choice([0.2, 0.1, 0.05])))]
            f.variants = G.variants_for(G.speeds_linear(int(shape.integers(4, 17))))
        elif kind == "running":
            f.team[f.passer, 0] = f.ball[0] = np.float32(shape.uniform(-6.0, 6.0))
            f.windows = front_zones(f.ball, G.Params())
        if "speeds" in case:
            f.variants = G.variants_for(_speeds(case), flat=True, chip=case["chip"])
        out.append(f)
    return out


def _params(case):
    return G.Params(n_samples=case.get("K", 64)).as_f32()


def _weights():
    with np.load(WEIGHTS, allow_pickle=False) as z:
        return np.ascontiguousarray(z["params"], np.float32)


def _targets(case, seed):
    """Training targets shaped like the exact score maps: a prior that grows
    toward the goal plus smooth noise, infeasible in connected regions."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    n = case["n"]
    cx = 0.2 * (torch.arange(61, device="cuda") - 30.0)
    cy = 0.2 * (torch.arange(46, device="cuda") - 22.5)
    prior = 0.3 * (1.0 - torch.hypot(cx[None, :] - 6.0, cy[:, None]) / 15.0)
    up = torch.nn.functional.interpolate
    smooth = up(torch.rand((n, 2, 10, 13), device="cuda", generator=g), size=(46, 61),
                mode="bilinear", align_corners=True)
    t = prior + 0.05 + 0.25 * smooth[:, 0]
    t = torch.where(smooth[:, 1] < 0.5, torch.full_like(t, -math.inf), t)
    return t.reshape(n, CELLS).contiguous()


def _records(t, dt, n):
    """The integer and float fields of device records, as views."""
    w = dt.itemsize // 4
    ints = sum(1 for name in dt.names if dt[name] == np.dtype("<i4") and name != "pad")
    stop = w - (1 if "pad" in dt.names else 0)
    t = t[:n * dt.itemsize]
    return (t.view(torch.int32).view(n, w)[:, :ints],
            t.view(torch.float32).view(n, w)[:, ints:stop])


_HOST_INTS = ("found", "window", "variant", "i", "j", "type")
_HOST_FLOATS = ("x", "y", "v0", "score", "t_team", "t_opp", "t_ball")


def _host_record(r):
    return [int(r[k]) for k in _HOST_INTS], np.array([r[k] for k in _HOST_FLOATS], np.float32)


def prepare(case, seed):
    kind = case["kind"]
    p = _params(case)
    flags = B.DPPS_OUT_REDUCED if case.get("reduced") else 0
    s = B.Searcher(p, out_flags=flags)
    frames = _frames(case, seed)
    st = {"case": case, "s": s, "kind": kind}
    if kind == "search":
        st["pk"] = B.pack(frames, p, flags)
        st["out"] = s.outputs_for(st["pk"])
    elif kind == "resident":
        st["batch"] = s.batch(frames)
        out = st["out"] = s.outputs_for(st["batch"].pk)
        st["batch"].autotune(out, reps=2)
        st["result"] = (out.mask, out.score, _records(out.best, B.BEST_DT, len(frames)))
    elif kind == "requests":
        st["pk"] = B.pack(frames, p, flags)
        out = st["out"] = s.outputs_for(st["pk"])
        st["result"] = (out.mask, out.score, _records(out.best, B.BEST_DT, len(frames)))
    elif kind == "sweep":
        pk = st["pk"] = B.pack(frames, p)
        total = case["dirs"] * int(pk.frames["n_variants"].sum())
        out = st["out"] = B.RayDeviceOutputs(total, len(frames), s.device)
        st["result"] = (out.mask, out.score, out.t_team, out.t_opp, out.s_recv,
                        _records(out.best, B.RAY_BEST_DT, len(frames)))
    elif kind == "power":
        st["frames"] = frames
    elif kind == "shot":
        pk = st["pk"] = s.pack_shots(frames, map=case["map"])
        it = B.SHOT_DT.itemsize
        ball = torch.zeros(len(frames) * it, dtype=torch.uint8, device=s.device)
        mp = torch.zeros(max(pk.total, 1) * it, dtype=torch.uint8, device=s.device)
        st["out"] = (ball, mp if case["map"] else None)
        st["result"] = [_records(ball, B.SHOT_DT, len(frames))]
        if case["map"]:
            st["result"].append(_records(mp, B.SHOT_DT, pk.total))
    elif kind == "running":
        pk = st["pk"] = B.pack(frames, p)
        n = int(pk.frames["n_windows"].sum())
        best = torch.zeros(n * B.RUN_BEST_DT.itemsize, dtype=torch.uint8, device=s.device)
        sc = torch.zeros(pk.total, dtype=torch.float32, device=s.device)
        st["out"] = (best, sc)
        st["result"] = (sc, _records(best, B.RUN_BEST_DT, n))
    else:
        n = case["n"]
        net = st["net"] = B.Mlp(s, n, max_k=case.get("k", 1))
        net.set_params(_weights())
        if kind == "proposals_host":
            st["pk"] = B.pack(frames, p)
            st["best"] = torch.zeros(n * B.BEST_DT.itemsize, dtype=torch.uint8, device=s.device)
            st["host"] = np.zeros(n, B.BEST_DT)
        else:
            st["batch"] = s.batch(frames)
        if kind == "forward":
            st["out"] = torch.empty((n, CELLS), dtype=torch.float32, device=s.device)
        elif kind == "train":
            st["target"] = _targets(case, seed)
        elif kind == "proposals":
            st["best"] = torch.zeros(n * B.BEST_DT.itemsize, dtype=torch.uint8, device=s.device)
            st["result"] = _records(st["best"], B.BEST_DT, n)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    kind, case, s = state["kind"], state["case"], state["s"]
    if kind == "search":
        out, best = s.search(state["pk"], out=state["out"])
        return out.mask, out.score, _host_record(best)
    if kind == "resident":
        state["batch"].run(state["out"], graph=True)
        return state["result"]
    if kind == "requests":
        s.search_batch(state["pk"], out=state["out"])
        return state["result"]
    if kind == "sweep":
        s.ray_search(state["pk"], case["dirs"], out=state["out"])
        return state["result"]
    if kind == "power":
        out, v0 = s.search_power(state["frames"])
        return (out.mask, out.score, out.t_team, out.t_opp, v0,
                _records(out.best, B.BEST_DT, case["n"]))
    if kind == "shot":
        s.shot(state["pk"], map=case["map"], out=state["out"])
        return state["result"]
    if kind == "running":
        s.running_points(state["pk"], out=state["out"])
        return state["result"]
    if kind == "forward":
        return state["net"].forward(state["batch"], out=state["out"])
    if kind == "train":
        net, loss = state["net"], None
        for k in range(case["steps"]):
            loss = net.train_step(state["batch"], state["target"], 3e-4, pos_weight=8.0,
                                  ce_weight=0.2, tau=0.02, want_loss=k == case["steps"] - 1)
        return loss, net.get_params()
    if kind == "proposals":
        _, fallbacks = state["net"].search(state["batch"], k=case["k"], best=state["best"])
        return state["result"], fallbacks
    _, fallbacks = state["net"].search_frames(state["pk"], k=case["k"], best=state["best"],
                                              host=state["host"])
    h = state["host"]
    return (np.stack([h[k] for k in _HOST_INTS]), np.stack([h[k] for k in _HOST_FLOATS]),
            fallbacks)


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------

_MLP_FLOPS = 2 * (66 * 512 + 2 * 512 * 512 + 512 * CELLS)
_MLP_BYTES = 2 * (66 * 512 + 2 * 512 * 512 + 512 * CELLS)


def work(case):
    """Inputs read once, outputs written once; operations of the method as
    the package's work model counts them."""
    kind, n = case["kind"], case.get("n", 1)
    per_frame = 16 * (case.get("n_team", 8) + case.get("n_opp", 8)) + 128
    if kind in ("search", "resident", "requests"):
        ev = fl = pts = 0
        for f in _frames(case, 0):
            e, x = FL.frame_work(f, case["K"])
            ev, fl, pts = ev + e, fl + x, pts + f.n_points()
        return {"bytes": 5 * (pts if case["reduced"] else ev) + n * per_frame, "flops": fl}
    if kind == "sweep":
        e, x = FL.ray_frame_work(_frames(dict(case, n=1), 0)[0], case["K"], case["dirs"], 0)
        return {"bytes": n * (17 * e + per_frame), "flops": n * x}
    if kind == "power":
        nx, ny = G.lattice_dims(case["h"])
        fl = FL.point_flops(case["n_team"] - 1 + case["n_opp"], case["n_opp"], case["K"], 1, 0)
        return {"bytes": n * (17 * nx * ny + per_frame), "flops": n * nx * ny * fl}
    if kind == "shot":
        nx, ny = G.lattice_dims(case["h"]) if case["map"] else (0, 0)
        pts = n * (1 + nx * ny)
        return {"bytes": 32 * pts + n * per_frame,
                "flops": pts * FL.shot_flops(case["n_opp"], case["K"])}
    if kind == "running":
        pts = sum(f.n_points() for f in _frames(case, 0))
        return {"bytes": 4 * pts + n * per_frame, "flops": pts * FL.run_flops(case["n_opp"])}
    if kind == "forward":
        return {"bytes": n * (4 * CELLS + per_frame) + _MLP_BYTES, "flops": n * _MLP_FLOPS}
    if kind == "train":
        # weights, moments and targets read, weights and moments written, per step
        return {"bytes": case["steps"] * (n * 4 * CELLS + 6 * 4 * _MLP_BYTES // 2),
                "flops": case["steps"] * n * 3 * _MLP_FLOPS}
    fine = 16 * case["k"] * FL.point_flops(case["n_team"] - 1 + case["n_opp"], case["n_opp"], 64,
                                           1, 0)
    return {"bytes": n * (56 + per_frame) + _MLP_BYTES, "flops": n * (_MLP_FLOPS + fine)}


# ---------------------------------------------------------------------------
# exact values: the method in float64, plain torch
# ---------------------------------------------------------------------------

def _d(x):
    return torch.as_tensor(np.asarray(x, np.float64), device="cuda")


def _points(p, w):
    h, i0, j0, nx, ny = float(np.float32(w[0])), *[int(v) for v in w[1:]]
    Nx, Ny = round(p.field_len / h) + 1, round(p.field_wid / h) + 1
    x = h * (i0 + torch.arange(nx, device="cuda", dtype=torch.float64) - 0.5 * (Nx - 1))
    y = h * (j0 + torch.arange(ny, device="cuda", dtype=torch.float64) - 0.5 * (Ny - 1))
    return torch.stack([x[None, :].expand(ny, nx), y[:, None].expand(ny, nx)], -1).reshape(-1, 2)


def _ball(p, typ, v0):
    """(stopping distance, first reachable distance, time to a distance)."""
    v0 = torch.as_tensor(v0, dtype=torch.float64, device="cuda")

    def phase(v, a, x):
        return 2 * x / (v + torch.sqrt(torch.clamp(v * v - 2 * a * x, min=0.0)))

    if typ == G.CHIP:
        vh, vz = v0 * math.cos(p.chip_angle), v0 * math.sin(p.chip_angle)
        tf = 2 * vz / p.gravity
        sf = vh * tf
        D = sf + vh * vh / (2 * p.roll_decel)
        return D, sf, lambda s: torch.where(s <= sf, s / vh, tf + phase(vh, p.roll_decel, s - sf))
    v1 = p.slide_ratio * v0
    t1, d1 = (v0 - v1) / p.slide_decel, (v0 * v0 - v1 * v1) / (2 * p.slide_decel)
    D = d1 + v1 * v1 / (2 * p.roll_decel)
    return D, torch.zeros_like(D), lambda s: torch.where(
        s <= d1, phase(v0, p.slide_decel, s), t1 + phase(v1, p.roll_decel, s - d1))


def _arrival(p, rob, pts):
    """Earliest arrival over the robots [R, 4] at the points [..., 2]."""
    A, V = p.amax, p.vmax
    best = torch.full(pts.shape[:-1], math.inf, dtype=torch.float64, device="cuda")
    for r in rob:
        d = pts - r[:2]
        rho = torch.linalg.vector_norm(d, dim=-1)
        dl = torch.clamp(rho - p.robot_radius, min=0.0)
        u = torch.where(rho > 0, (d * r[2:]).sum(-1) / torch.where(rho > 0, rho, 1.0), 0.0)
        u = torch.clamp(u, -V, V)
        ss = u * u / (2 * A)
        back = (u >= 0) & (ss >= dl)
        D = torch.where(back, ss - dl, ss + dl)
        rest = torch.where(D >= V * V / A, D / V + V / A, 2 * torch.sqrt(D / A))
        best = torch.minimum(best, torch.where(back, u / A, -u / A) + rest)
    return best


def _mouth(p, c):
    dx = torch.clamp(p.goal_x - c[:, 0], min=p.goal_eps)
    return (torch.atan2(-0.5 * p.goal_width - c[:, 1], dx),
            torch.atan2(0.5 * p.goal_width - c[:, 1], dx))


def _shadows(p, c, opp):
    """Sorted shadow intervals [n, o] clipped to the mouth, and who is inside."""
    lo, hi = _mouth(p, c)
    o = opp[None, :, :2] - c[:, None]
    rho = torch.linalg.vector_norm(o, dim=-1)
    front = (opp[:, 0] < p.goal_x)[None]
    al = torch.asin(torch.clamp(p.robot_radius / torch.clamp(rho, min=1e-12), max=1.0))
    phi = torch.atan2(o[..., 1], o[..., 0])
    s, e = torch.maximum(phi - al, lo[:, None]), torch.minimum(phi + al, hi[:, None])
    has = front & (e > s)
    s, e = torch.where(has, s, hi[:, None]), torch.where(has, e, hi[:, None])
    s, order = torch.sort(s, dim=-1)
    e = torch.gather(e, -1, order)
    inside = (front & (rho <= p.robot_radius)).any(-1)
    return lo, hi, s, e, inside


def _gaps(p, c, opp):
    """(widths, starts) of the open gaps in increasing angle."""
    lo, hi, s, e, inside = _shadows(p, c, opp)
    edge = torch.cummax(torch.cat([lo[:, None], e], -1), -1).values
    w = torch.clamp(torch.cat([s, hi[:, None]], -1) - edge, min=0.0)
    return torch.where(inside[:, None], 0.0, w), edge


def _score(p, c, opp, m):
    ang = _gaps(p, c, opp)[0].sum(-1)
    dist = torch.hypot(c[:, 0] - p.goal_x, c[:, 1])
    base = p.w_angle * ang / math.pi + p.w_dist * (1 - dist / p.dist_norm)
    return base[:, None] + p.w_margin * torch.clamp(m, 0.0, p.margin_cap_s)


def _first(allowed, T, tb):
    return torch.where(allowed & (T <= tb), tb, math.inf).amin(-1)


def _margin(tt, to):
    return torch.where(torch.isfinite(tt), torch.where(torch.isfinite(to), to - tt, math.inf),
                       -math.inf)


def _sides(f):
    team = np.delete(np.asarray(f.team, np.float64), f.passer, 0)
    return _d(team.reshape(-1, 4)), _d(np.asarray(f.opp, np.float64).reshape(-1, 4))


def _search64(p, f, pts, variants, speed=None):
    """Scores, times [n, variants] of candidate points; with speed, one flat
    pass per point at speed(points)."""
    team, opp = _sides(f)
    b = _d(f.ball)
    K = p.n_samples
    frac = (torch.arange(K, device="cuda", dtype=torch.float64) + 1) / K
    outs = []
    for c in pts.split(max(1, 4_000_000 // K)):
        d = torch.linalg.vector_norm(c - b, dim=-1)
        path = b + frac[None, :, None] * (c - b)[:, None]
        Tt, To = _arrival(p, team, path), _arrival(p, opp, path)
        s = frac[None] * d[:, None]
        tts, tos, vs = [], [], []
        for typ, v0 in ([(G.FLAT, None)] if speed else variants):
            if speed:
                v0 = speed(c, d)
                vs.append(v0)
                D, sf, t = _ball(p, typ, v0[:, None])
                D, sf = D[:, 0], sf[:, 0]
            else:
                D, sf, t = _ball(p, typ, v0)
            reach = (d >= 1e-9) & (d <= D) & (d >= sf)
            tb = t(s)
            ok = reach[:, None] & (s >= (sf[:, None] if sf.dim() else sf))
            tts.append(_first(ok, Tt, tb))
            tos.append(_first(ok, To, tb))
        tt, to = torch.stack(tts, -1), torch.stack(tos, -1)
        m = _margin(tt, to)
        sc = torch.where(m >= p.margin_s, _score(p, c, opp, m), -math.inf)
        outs.append((sc, tt, to) + ((torch.stack(vs, -1),) if speed else ()))
    return [torch.cat(x) for x in zip(*outs)]


def _exact_maps(case, seed):
    p = _params(case)
    got = []
    for f in _frames(case, seed):
        for w in f.windows:
            sc = _search64(p, f, _points(p, w), f.variants)[0]
            got.append(sc.amax(-1) if case["reduced"] else sc.t().reshape(-1))
    return None, torch.cat(got), None


def _exact_power(case, seed):
    p = _params(case)
    got = []
    for f in _frames(case, seed):
        team, _ = _sides(f)

        def speed(c, d, team=team):
            t = _arrival(p, team, c) + float(np.float32(0.3))
            a = p.roll_decel
            v1 = torch.where(d >= 0.5 * a * t * t, (d + 0.5 * a * t * t) / t,
                             torch.sqrt(2 * a * d))
            return torch.clamp(v1 / p.slide_ratio, 1.0, 6.5)

        got.append(_search64(p, f, _points(p, f.windows[0]), None, speed))
    sc, tt, to, v0 = [torch.cat([x[:, 0] for x in g]) for g in zip(*got)]
    return None, sc, tt, to, v0, None


def _exact_sweep(case, seed):
    p = _params(case)
    n_dirs, K = case["dirs"], case["K"]
    th = 2 * math.pi * torch.arange(n_dirs, device="cuda", dtype=torch.float64) / n_dirs
    u = torch.stack([torch.cos(th), torch.sin(th)], -1)
    frac = (torch.arange(K, device="cuda", dtype=torch.float64) + 1) / K
    half = _d([p.field_len / 2, p.field_wid / 2])
    got = []
    for f in _frames(case, seed):
        team, opp = _sides(f)
        b = _d(f.ball)
        L = torch.where(u.abs() > 1e-15, (torch.sign(u) * half - b) / u, math.inf)
        L = torch.clamp(L.amin(-1), min=0.0)
        s = frac[None] * L[:, None]
        path = b + s[..., None] * u[:, None]
        Tt, To = _arrival(p, team, path), _arrival(p, opp, path)
        cols = []
        for typ, v0 in f.variants:
            D, sf, t = _ball(p, typ, v0)
            tb, ok = t(s), (s <= D) & (s >= sf)
            tt, to = _first(ok, Tt, tb), _first(ok, To, tb)
            sr = torch.where(ok & (Tt <= tb), s, math.inf).amin(-1)
            m = _margin(tt, to)
            c = b + torch.where(torch.isfinite(sr), sr, 0.0)[:, None] * u
            g = _d([p.goal_x, 0.0]) - c
            ref = torch.atan2((u[:, 0] * g[:, 1] - u[:, 1] * g[:, 0]).abs(), (u * g).sum(-1))
            sc = (_score(p, c, opp, m[:, None])[:, 0] - 0.05 * tt - 0.1 * ref / math.pi)
            cols.append((torch.where(m >= p.margin_s, sc, -math.inf), tt, to, sr))
        got.append([torch.stack(x, -1).reshape(-1) for x in zip(*cols)])
    return (None, *[torch.cat(x) for x in zip(*got)], None)


def _shot64(p, opp, c):
    """Float fields of the shooting decision from the points c [n, 2]."""
    w, start = _gaps(p, c, opp)
    gap, k = w.max(-1)
    dx = torch.clamp(p.goal_x - c[:, 0], min=p.goal_eps)
    aim = torch.where(gap > 0, start.gather(-1, k[:, None])[:, 0] + 0.5 * gap,
                      torch.atan2(-c[:, 1], dx))
    L = dx / torch.cos(aim)
    D, _, t = _ball(p, G.FLAT, 6.5)
    K = p.n_samples
    frac = (torch.arange(K, device="cuda", dtype=torch.float64) + 1) / K
    s = frac[None] * L[:, None]
    u = torch.stack([torch.cos(aim), torch.sin(aim)], -1)
    T = _arrival(p, opp, c[:, None] + s[..., None] * u[:, None])
    slack = torch.where(s <= D, T - t(s), math.inf).amin(-1)
    t_goal = torch.where(L <= D, t(L), math.inf)
    return torch.stack([aim, gap, w.sum(-1), L, t_goal, slack], -1)


def _exact_shot(case, seed):
    p = _params(case)
    ball, maps = [], []
    for f in _frames(case, seed):
        opp = _sides(f)[1]
        ball.append(_shot64(p, opp, _d(f.ball)[None]))
        if case["map"]:
            maps += [_shot64(p, opp, c) for c in _points(p, f.windows[0]).split(8192)]
    out = [(None, torch.cat(ball))]
    return out + [(None, torch.cat(maps))] if case["map"] else out


def _exact_running(case, seed):
    p = _params(case)
    R = {k: float(np.float32(v)) for k, v in B.RUN_DEFAULTS.items()}
    x0, hw = p.goal_x - R["def_depth"], 0.5 * R["def_width"]
    got = []
    for f in _frames(case, seed):
        opp = _sides(f)[1]
        b = _d(f.ball)
        c = torch.cat([_points(p, w) for w in f.windows])
        cx, cy = c[:, 0], c[:, 1]
        gx, gy = p.goal_x - cx, -cy
        x1 = 1 - torch.hypot(gx, gy) / p.dist_norm
        db = torch.linalg.vector_norm(c - b, dim=-1)
        x2 = torch.clamp(db / R["ball_norm"], max=1.0)
        phi = torch.atan2(gy, gx).abs()
        off = torch.clamp(R["ang_lo"] - phi, min=0.0) + torch.clamp(phi - R["ang_hi"], min=0.0)
        x3 = torch.clamp(1 - off / R["ang_fall"], min=0.0)
        guard = 0.0
        for post in (0.5 * p.goal_width, -0.5 * p.goal_width):
            dy = post - cy
            tx = torch.where(gx != 0, (torch.where(gx > 0, x0, p.goal_x) - cx)
                             / torch.where(gx != 0, gx, 1.0), 0.0)
            ty = torch.where(dy != 0, (torch.where(dy > 0, -hw, hw) - cy)
                             / torch.where(dy != 0, dy, 1.0), 0.0)
            t = torch.clamp(torch.maximum(tx, ty), 0.0, 1.0)
            guard = guard + _arrival(p, opp, torch.stack([cx + t * gx, cy + t * dy], -1))
        x4 = torch.clamp(guard / R["guard_norm"], max=1.0)
        near = torch.linalg.vector_norm(opp[:, :2] - b, dim=-1)[None] < db[:, None]
        away = torch.linalg.vector_norm(opp[None, :, :2] - c[:, None], dim=-1)
        x5 = 1 - torch.where(near, torch.clamp(1 - away / R["mark_radius"], min=0.0), 0.0).amax(-1)
        sc = (R["w_goal"] * x1 + R["w_ball"] * x2 + R["w_angle"] * x3 + R["w_guard"] * x4
              + R["w_defense"] * x5)
        out = (cx > x0) & (cx < p.goal_x) & (cy.abs() < hw)
        got.append(torch.where(out, -math.inf, sc))
    return torch.cat(got), None


def _features64(case, seed):
    p = _params(case)
    rows = []
    for f in _frames(case, seed):
        x = np.zeros(66)
        ball = np.asarray(f.ball, np.float64)
        for side, rob in enumerate((f.team, f.opp)):
            rob = np.asarray(rob, np.float64).reshape(-1, 4)
            key = ((rob[:, :2] - ball) ** 2).sum(1)
            if side == 0:
                key[f.passer] = -1.0
            rob = rob[np.argsort(key, kind="stable")[:8]]
            x[32 * side:32 * side + 4 * len(rob)] = (rob / [6.0, 4.5, p.vmax, p.vmax]).reshape(-1)
        x[64:] = ball / [6.0, 4.5]
        rows.append(x)
    return _d(np.stack(rows))


def _layers64(flat):
    flat, out, o = _d(flat), [], 0
    for r, c in ((512, 66), (512, 512), (512, 512), (CELLS, 512)):
        out += [flat[o:o + r * c].view(r, c).clone(), flat[o + r * c:o + r * c + r].clone()]
        o += r * c + r
    return out


def _net64(par, x):
    for k in range(0, 8, 2):
        x = x @ par[k].t() + par[k + 1]
        if k < 6:
            x = torch.nn.functional.gelu(x)
    return x


def _exact_train(case, seed):
    par = [t.requires_grad_() for t in _layers64(_weights())]
    opt = torch.optim.Adam(par, lr=3e-4, betas=(0.9, 0.999), eps=1e-8)
    x, raw = _features64(case, seed), _targets(case, seed).double()
    t = torch.where(torch.isfinite(raw), raw, 0.0)
    q = torch.softmax(raw / 0.02, -1)
    loss = None
    for _ in range(case["steps"]):
        opt.zero_grad()
        y = _net64(par, x)
        ce = -(q * torch.log_softmax(y / 0.02, -1)).sum(-1).mean()
        loss = ((1 + 8.0 * t) * (y - t) ** 2).mean() + 0.2 * ce
        loss.backward()
        opt.step()
    return float(loss), torch.cat([w.detach().reshape(-1) for w in par])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("search", "resident", "requests"):
        return _exact_maps(case, seed)
    if kind == "sweep":
        return _exact_sweep(case, seed)
    if kind == "power":
        return _exact_power(case, seed)
    if kind == "shot":
        return _exact_shot(case, seed)
    if kind == "running":
        return _exact_running(case, seed)
    if kind == "forward":
        return _net64(_layers64(_weights()), _features64(case, seed))
    if kind == "train":
        return _exact_train(case, seed)
    return None  # chosen passes: indices, with the exact search's own scores
