"""Performance cases: the evaluations that a program asks of this library.

Each case goes through the public calls of ``paper_2604_27193_amd.binding``.
``listed()`` names the fixed ones, ``draw()`` gives others of the same ranges,
``prepare()`` builds what a program holds before the call, ``run()`` is one
pass, ``work()`` the least bytes and operations of a pass, and ``exact()`` the
outputs in 64 bits by plain torch, step by step, sharing no code with the
library.

A case is a dict: ``kind`` (which evaluation), ``n`` (samples, of each scenario
in a batch), ``precision`` and the scenario's options.  Kinds:

* ``plain``   parameter columns in device memory, rollout, statistics
* ``request`` parameters drawn in the kernel, rollout, statistics
* ``graph``   as ``plain``, recorded once and replayed
* ``sweep``   a grid of lead-vehicle scenarios in one batched launch, then the
              statistics of each
* ``uneven``  scenarios of uneven sizes, horizons and steps as one recorded
              batch, replayed
* ``serve``   requests submitted to the server at once and collected
"""
import time

import numpy as np
import torch

from paper_2604_27193_amd import binding as B
from paper_2604_27193_amd import workloads as W

DEV = "cuda"
# headways at three risk levels, two margin quantiles and a risk curve: the
# statistics of an assessment
REQ = {"risk": (0.05, 0.01, 0.001), "margin_q": (0.01, 0.05), "grid": (20.0, 140.0, 121)}
SERVE_SIZES = ((25_000, 0.70), (100_000, 0.25), (1_000_000, 0.05))
FLOATS = ("dist", "margin", "v_impact")


def listed():
    return [
        # the smallest call: one quick estimate, where launches and latency count
        {"name": "request_1k", "kind": "request", "model": "single", "n": 1000,
         "precision": "fp64", "dt": 1e-3},
        # the real-time request: 25,000 samples within the 530 ms budget
        {"name": "request_25k", "kind": "request", "model": "single", "n": 25_000,
         "precision": "fp64", "dt": 1e-3},
        # the same size as a steady loop: columns refilled by the caller, one
        # recorded launch per evaluation; a ragged size
        {"name": "graph_25k_fp32c", "kind": "graph", "model": "single", "n": 25_013,
         "precision": "fp32c", "dt": 1e-3},
        # the plain method at full size: columns in device memory, FP64
        {"name": "plain_1m_fp64", "kind": "plain", "model": "single", "n": 1_048_576,
         "precision": "fp64", "dt": 1e-3},
        # the served form at full size: drawn in the kernel, compensated FP32
        {"name": "request_1m_fp32c", "kind": "request", "model": "single", "n": 1_048_576,
         "precision": "fp32c", "dt": 1e-3},
        # the paper's preset with its integrator, the largest row of its table
        {"name": "paper_rk4_350k", "kind": "request", "model": "paper", "n": 350_000,
         "precision": "fp64", "dt": 1e-3},
        # rare events: the preset with shifted proposals and weighted statistics
        {"name": "rare_rk4_1m", "kind": "request", "model": "rare", "n": 1_048_576,
         "precision": "fp64", "dt": 1e-3},
        # perception delays differ between samples
        {"name": "perception_200k", "kind": "request", "model": "perception", "n": 200_003,
         "precision": "fp64", "dt": 1e-3},
        # a cell of the controller assessment
        {"name": "closed_loop_200k", "kind": "request", "model": "closed_loop", "n": 200_000,
         "precision": "fp64", "dt": 1e-3},
        # the scenario sweep: 256 lead-vehicle scenarios of 100,000 samples, the largest
        {"name": "sweep_lead_fp32c", "kind": "sweep", "side": 16, "n": 100_000,
         "precision": "fp32c", "dt": 1e-3},
        # 1,000 uneven scenarios as one recorded batch
        {"name": "uneven_1000_fp32c", "kind": "uneven", "scenarios": 1000, "n": 100_000,
         "precision": "fp32c"},
        # a burst of requests of mixed sizes at the server
        {"name": "serve_mix_fp32c", "kind": "serve", "requests": 40, "precision": "fp32c"},
    ]


def _log_int(rng, lo, hi):
    n = int(round(lo * (hi / lo) ** rng.random()))
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(("request", "request", "request", "plain", "plain", "graph", "sweep",
                       "sweep", "uneven", "serve"))
    if kind == "sweep":
        return {"kind": kind, "side": rng.choice((2, 3, 5, 8, 16)),
                "n": _log_int(rng, 1000, 40_000), "precision": rng.choice(("fp64", "fp32c")),
                "dt": rng.choice((1e-3, 2e-3))}
    if kind == "uneven":
        return {"kind": kind, "scenarios": _log_int(rng, 3, 500),
                "n": _log_int(rng, 5000, 100_000), "precision": rng.choice(("fp64", "fp32c"))}
    if kind == "serve":
        return {"kind": kind, "requests": _log_int(rng, 1, 60),
                "precision": rng.choice(("fp64", "fp32c"))}
    model = rng.choice(("single", "single", "paper", "paper", "rare", "perception",
                        "closed_loop", "lead"))
    if kind != "request" and model == "rare":
        model = "paper"
    c = {"kind": kind, "model": model, "n": _log_int(rng, 1000, 1_048_576), "precision": "fp64",
         "dt": rng.choice((0.5e-3, 1e-3, 1e-3, 2e-3))}
    if model in ("single", "perception", "lead"):
        c["precision"] = rng.choice(("fp64", "fp64", "fp32c", "fp32c_fixup"))
        if c["precision"] == "fp64" and rng.random() < 0.2:
            c["nofma"] = True
        if model == "single" and rng.random() < 0.25:
            c["impact_exit"] = True
    if model == "paper" and rng.random() < 0.3:
        c["integrator"] = "euler"
        c["precision"] = rng.choice(("fp64", "fp32c"))
    return c


# ---- scenarios ----

def _one(case, seed):
    over = {"dt": case["dt"]}
    for f in ("nofma", "impact_exit"):
        if case.get(f):
            over[f] = True
    n, m = case["n"], case["model"]
    if m == "single":
        return W.single(n, seed=seed, **over)
    if m == "perception":
        return W.perception(n, seed=seed, **over)
    if m == "closed_loop":
        return W.closed_loop(n, seed=seed, **over)
    if m == "paper":
        return W.paper_preset(n, seed=seed, integrator=case.get("integrator", "rk4"), **over)
    if m == "rare":
        return W.rare_event(n, seed=seed, **over)
    # one cell of the sweep: a lead vehicle braking at N(3, 0.5) from N(40, 3)
    return W.single(n, seed=seed, obstacle="lead", gap=("normal", 40.0, 3.0),
                    lead_decel=("normal", 3.0, 0.5), **over)


def _scenarios(case, seed):
    k = case["kind"]
    if k == "sweep":
        s = case["side"]
        out = W.sweep(case["n"], seed=seed, v0_means=np.linspace(10.0, 40.0, s),
                      mu_means=np.linspace(0.2, 1.0, s))
        for d in out:
            d["dt"] = case["dt"]
        return out
    if k == "uneven":
        # the sizes, horizons and steps of the configuration; the seed draws the samples
        out = W.uneven_batch(case["scenarios"], max_samples=case["n"])
        for d in out:
            d["seed"] = seed
        return out
    if k == "serve":
        rng = np.random.Generator(np.random.PCG64(seed))
        m = case["requests"]
        sizes = [SERVE_SIZES[0][0]] * m
        at = 0
        for n, share in SERVE_SIZES[1:]:
            for _ in range(int(m * share)):
                sizes[at] = n
                at += 1
        sizes = rng.permutation(sizes)
        reqs = W.serving_stream(800, duration=1.0, seed=seed)[:m]
        out = []
        for (_, d, _), n in zip(reqs, sizes):
            d["n_samples"] = int(n)
            out.append(d)
        return out
    return [_one(case, seed)]


# ---- the pass ----

def _outs(scns):
    """Output columns of all the scenarios side by side, and each one's part."""
    total = sum(d["n_samples"] for d in scns)
    whole = B.alloc_outputs(total, weight=bool(scns[0].get("proposal")))
    parts, at = [], 0
    for d in scns:
        parts.append({k: v[at:at + d["n_samples"]] for k, v in whole.items()})
        at += d["n_samples"]
    return whole, parts


def prepare(case, seed):
    scns = _scenarios(case, seed)
    st = {"case": case, "scns": scns}
    k = case["kind"]
    if k == "serve":
        # the launches' own memory, and room for every request of the burst
        need = B.Server.fixed_bytes(case["precision"], n_streams=2, **REQ) + 2 ** 30
        st["server"] = B.Server(need, precision=case["precision"], n_streams=2, **REQ)
        return st
    st["whole"], st["parts"] = _outs(scns)
    if k in ("plain", "graph"):
        st["params"] = _draw(scns[0])
    if k == "graph":
        st["graph"] = B.Graph(scns[0], params=st["params"], precision=case["precision"],
                              out=st["parts"][0], **REQ)
    if k == "uneven":
        st["graph"] = B.Graph(scns, precision=case["precision"], out=st["parts"], batch=True,
                              **REQ)
    return st


def _stats(s):
    """The statistics of several scenarios as arrays, one row each."""
    return {k: np.array([x[k] for x in s]) for k in s[0]}


def run(state):
    k = state["case"]["kind"]
    prec = state["case"]["precision"]
    scns = state["scns"]
    if k == "serve":
        srv = state["server"]
        tickets = [srv.submit(d) for d in scns]
        res = []
        for t in tickets:
            r = srv.poll(t)
            while r is None:
                time.sleep(2e-5)
                r = srv.poll(t)
            res.append(r[0])
        return {"stats": _stats(res)}
    if k in ("graph", "uneven"):
        state["graph"].launch()
        s = state["graph"].finish()
        s = s if k == "uneven" else [s]
    elif k == "sweep":
        B.batch_rollout(scns, precision=prec, outs=state["parts"])
        s = B.batch_reduce(state["parts"], **REQ)
    else:
        B.rollout(scns[0], params=state.get("params"), precision=prec, out=state["parts"][0])
        s = [B.reduce(state["parts"][0], **REQ)]
    return {**state["whole"], "stats": _stats(s)}


# Mean time to the end of a rollout (s) of each model, and the operations of
# one step: explicit Euler 11 (9 in the compensated form; a lead vehicle adds
# 7), classical RK4 57.
MEAN_T = {"single": 4.87, "perception": 5.14, "closed_loop": 7.25, "paper": 5.16, "rare": 7.49,
          "lead": 4.8}


def work(case):
    k = case["kind"]
    fp32 = case["precision"] != "fp64"
    per = 9.0 if fp32 else 11.0
    if k == "sweep":
        n = case["side"] ** 2 * case["n"]
        steps = n * 5.53 / case["dt"]
        per += 7.0
    elif k == "uneven":
        # log-uniform sizes in [1e3, 1e6], capped; steps of 0.5, 1 and 2 ms
        c = np.log(case["n"] / 1e3) / np.log(1e3)
        n = case["scenarios"] * ((case["n"] - 1e3) / np.log(1e3) + (1.0 - c) * case["n"])
        steps = n * 4.68 * (2000 + 1000 + 500) / 3
    elif k == "serve":
        m = case["requests"]
        n = sum(s * int(m * p) for s, p in SERVE_SIZES[1:])
        n += SERVE_SIZES[0][0] * (m - sum(int(m * p) for _, p in SERVE_SIZES[1:]))
        steps = n * 4.7e3
    else:
        n = case["n"]
        steps = n * MEAN_T[case["model"]] / case["dt"]
        if case["model"] in ("paper", "rare") and case.get("integrator", "rk4") == "rk4":
            per = 57.0
        elif case["model"] == "lead":
            per += 7.0
    moved = 0 if k == "serve" else 25 * n  # the five output columns
    if k in ("plain", "graph"):
        moved += 72 * n  # nine parameter columns
    return {"bytes": float(moved + 4096), "flops": float(per * steps)}


# ---- the same in 64 bits, by plain torch ----

_M32 = 0xFFFFFFFF
_SLOTS = ("v0", "mu", "mass", "grade", "cda", "crr", "tau", "gap", "lead_decel")


def _uniforms(seed, sid, n, slot, attempt=0):
    """Two uniforms per sample of Philox4x32-10 (Salmon et al., SC'11): counter
    (i, slot | attempt << 8, id), key seed; the top 52 bits of each half."""
    c0 = torch.arange(n, dtype=torch.int64, device=DEV)
    c1 = torch.full_like(c0, slot | (attempt << 8))
    c2 = torch.full_like(c0, sid & _M32)
    c3 = torch.full_like(c0, (sid >> 32) & _M32)
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        pa, pb = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64
        c0, c1, c2, c3 = (((pb >> 32) & _M32) ^ c1 ^ k0, pb & _M32,
                          ((pa >> 32) & _M32) ^ c3 ^ k1, pa & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    a, b = (c1 << 20) | (c0 >> 12), (c3 << 20) | (c2 >> 12)
    return (a.double() + 0.5) * 2.0 ** -52, (b.double() + 0.5) * 2.0 ** -52


def _normals(seed, sid, n, slot, attempt=0):
    a, b = _uniforms(seed, sid, n, slot, attempt)
    r, th = torch.sqrt(-2.0 * torch.log(a)), 6.283185307179586 * b
    return r * torch.cos(th), r * torch.sin(th)


def _dist(spec, d, n, slot):
    seed, sid = d["seed"], d["scenario_id"]
    if spec[0] == "const":
        return torch.full((n,), float(spec[1]), dtype=torch.float64, device=DEV)
    if spec[0] == "uniform":
        return spec[1] + (spec[2] - spec[1]) * _uniforms(seed, sid, n, slot)[0]
    x = spec[1] + spec[2] * _normals(seed, sid, n, slot)[0]
    if spec[0] == "normal":
        return x
    lo, hi = spec[3], spec[4]
    for j in range(1, 16):
        out = (x < lo) | (x > hi)
        if not bool(out.any()):
            break
        x = torch.where(out, spec[1] + spec[2] * _normals(seed, sid, n, slot, j)[0], x)
    return x.clamp(lo, hi)


def _trigger(d, n):
    """Perception: the delay of each sample's brake request."""
    lat = _dist(d["latency"], d, n, 9).clamp(min=0.0)
    per = d["frame_period"]
    if per == 0.0:
        return lat
    hidden = torch.floor(_dist(d["occlusion"], d, n, 10).clamp(min=0.0))
    t = torch.full((n,), float("inf"), dtype=torch.float64, device=DEV)
    row = torch.zeros(n, dtype=torch.int64, device=DEV)
    u = None
    for j in range(int(np.floor(d["horizon"] / per)) + 1):
        if j % 2 == 0:
            u = _uniforms(d["seed"], d["scenario_id"], n, 11, j // 2)
        seen = (u[j % 2] >= d["p_dropout"]) & (hidden <= j)
        row = torch.where(seen, row + 1, torch.zeros_like(row))
        t = torch.where((row >= d["confirm"]) & torch.isinf(t), j * per + lat, t)
        if j % 8 == 7 and not bool(torch.isinf(t).any()):
            break
    return t


def _draw(d):
    """The parameter columns of a scenario's samples."""
    n = d["n_samples"]
    prop = d.get("proposal", {})
    p, lw = {}, torch.zeros(n, dtype=torch.float64, device=DEV)
    for slot, f in enumerate(_SLOTS):
        x = _dist(prop.get(f, d[f]), d, n, slot)
        if f in prop:
            zp, zq = (x - d[f][1]) / d[f][2], (x - prop[f][1]) / prop[f][2]
            lw += np.log(prop[f][2] / d[f][2]) + 0.5 * zq * zq - 0.5 * zp * zp
        p[f] = x
    p["sin_grade"], p["cos_grade"] = torch.sin(p["grade"]), torch.cos(p["grade"])
    if "latency" in d:
        p["trigger"] = _trigger(d, n)
    if prop:
        p["log_weight"] = lw
    return p


def _rollout(d, p):
    """Every sample's rollout, one step at a time."""
    n, dt = d["n_samples"], d["dt"]
    nmax = int(round(d["horizon"] / dt))
    kd = 0.5 * d["rho"] * p["cda"] / p["mass"]
    c = d["g"] * p["sin_grade"] + p["crr"] * d["g"] * p["cos_grade"]
    alim = -(p["mu"] * d["g"] / (1.0 + p["mu"] * d["h_cog"] / d["wheelbase"]))
    lead, ctl = d["obstacle"] == "lead", d.get("ctl_period", 0.0) > 0.0
    obs = d["obstacle"] != "none"
    exits = lead or d.get("impact_exit", False)
    zero = torch.zeros(n, dtype=torch.float64, device=DEV)
    trig = p.get("trigger", zero)
    nd = torch.round((d["dead_time"] + trig) / dt).clamp(max=float(nmax))
    nd_lo, nd_hi = int(nd.min()), int(nd.max())
    x, v, a = zero.clone(), p["v0"].clone(), zero.clone()
    xl, vl = zero.clone(), p["v0"].clone()
    gap, decel = p["gap"], p["lead_decel"]
    margin, vimp, dist, xmax = gap.clone(), zero.clone(), zero.clone(), zero.clone()
    hit = torch.zeros(n, dtype=torch.bool, device=DEV)
    live = ~hit
    stage = torch.zeros(n, dtype=torch.int64, device=DEV)
    start = [torch.full((n,), 2 ** 40, dtype=torch.int64, device=DEV) for _ in range(2)]
    per = int(round(d["ctl_period"] / dt)) if ctl else 0

    def slope(v_, a_):
        return torch.maximum(a_, alim) - kd * (v_ * v_) - c

    for k in range(nmax):
        if ctl:
            if k % per == 0:
                zg, zv = _normals(d["seed"], d["scenario_id"], n, 12, k // per)
                g = (gap + xl if lead else gap) - x + d["noise_gap"] * zg
                w = v - (vl if lead else 0.0) + d["noise_v"] * zv
                ttc = torch.where(w > 0.0, g / w, torch.full_like(w, float("inf")))
                want = (ttc < d["ttc_warn"]).long()
                want = torch.where(ttc < d["ttc_brake"], 2, want)
                for s in (1, 2):
                    up = (want == s) & (stage < s)
                    start[s - 1] = torch.where(up, k + int(round(d["dead_time"] / dt)),
                                               start[s - 1])
                    stage = torch.where(up, s, stage)
            cmd = torch.where(start[1] <= k, d["a_cmd"],
                              torch.where(start[0] <= k, d["a_warn"], 0.0))
        elif k < nd_lo:
            cmd = 0.0
        elif k >= nd_hi:
            cmd = d["a_cmd"]
        else:
            cmd = torch.where(nd <= k, d["a_cmd"], 0.0)
        if d["integrator"] == "rk4":
            k1 = slope(v, a)
            b1 = (cmd - a) / p["tau"]
            v2, a2 = v + 0.5 * dt * k1, a + 0.5 * dt * b1
            k2, b2 = slope(v2, a2), (cmd - a2) / p["tau"]
            v3, a3 = v + 0.5 * dt * k2, a + 0.5 * dt * b2
            k3, b3 = slope(v3, a3), (cmd - a3) / p["tau"]
            v4, a4 = v + dt * k3, a + dt * b3
            k4, b4 = slope(v4, a4), (cmd - a4) / p["tau"]
            x = x + dt / 6.0 * (v + 2.0 * v2 + 2.0 * v3 + v4)
            v = v + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
            a = a + dt / 6.0 * (b1 + 2.0 * b2 + 2.0 * b3 + b4)
        else:
            acc = slope(v, a)
            a = a + dt / p["tau"] * (cmd - a)
            x = x + dt * v
            v = v + dt * acc
        if lead:
            xl = xl + dt * vl
            vl = (vl - dt * decel).clamp(min=0.0)
        room = (gap + xl if lead else gap) - x
        margin = torch.where(live, torch.minimum(margin, room), margin)
        ends = v <= 0.0
        if obs:
            now = live & (room < 0.0) & ~hit
            vimp = torch.where(now, v - vl if lead else v, vimp)
            hit |= now
            if exits:
                ends = ends | hit
        if k + 1 == nmax:
            ends = torch.ones_like(ends)
        ends = ends & live
        dist = torch.where(ends, x, dist)
        # the distance at the horizon is no stop: kept for the statistics
        if k + 1 == nmax:
            xmax = torch.where(ends & (v > 0.0) & ~(hit if exits else torch.zeros_like(hit)),
                               1.0, 0.0)
        live = live & ~ends
        if k % 64 == 63 and not bool(live.any()):
            break
    return {"dist": dist, "margin": margin, "v_impact": torch.where(hit, vimp, zero),
            "hit": hit, "stop": (xmax == 0.0) & ~(hit if exits else torch.zeros_like(hit))}


def _statistics(r):
    """The float statistics of one scenario that counts and order give."""
    n = r["dist"].numel()
    d = torch.where(r["stop"], r["dist"], torch.full_like(r["dist"], float("inf")))
    s = torch.sort(d).values
    m = torch.sort(r["margin"]).values
    stop = r["dist"][r["stop"]]
    lo, hi, ng = REQ["grid"]
    grid = lo + torch.arange(ng, dtype=torch.float64, device=DEV) * ((hi - lo) / (ng - 1))
    over = n - torch.searchsorted(s, grid, right=True)
    return {"p_collision": float(r["hit"].double().mean()),
            "mean_dist": float(stop.mean()) if stop.numel() else float("nan"),
            "sd_dist": float(stop.std()) if stop.numel() > 1 else float("nan"),
            "headway": [float(s[n - int(np.floor(q * n)) - 1]) for q in REQ["risk"]],
            "margin_min": float(m[0]), "margin_mean": float(m.mean()),
            "margin_q": [float(m[int(np.floor(q * n))]) for q in REQ["margin_q"]],
            "risk_p": (over.double() / n).cpu().numpy()}


def exact(case, seed):
    scns = _scenarios(case, seed)
    # about 20 seconds at most
    if (sum(d["n_samples"] for d in scns) > 2_000_000
            or sum(d["horizon"] / d["dt"] for d in scns) > 100_000):
        return None
    got = [_rollout(d, _draw(d)) for d in scns]
    out = {"stats": _stats([_statistics(r) for r in got])}
    if case["kind"] != "serve":
        for f in FLOATS:
            out[f] = torch.cat([r[f] for r in got])
        if scns[0].get("proposal"):
            out["weight"] = torch.exp(torch.cat([_draw(d)["log_weight"] for d in scns]))
    return out
