"""The workloads whose time this framework is judged by, each through the public entry points.

A case is a dict of plain values; `prepare` builds its inputs on the GPU, `run` takes one
pass over them, `exact` gives the same outputs from plain float64 torch.  Kinds of passes:

  run      one simulation job on a kept Engine: admit the initial state, step to the horizon,
           read the per-step history, retire (the state at the last integer step comes back).
           A job starts from the same state every pass, so a pass is always the same physics.
  sweep    many uneven instances in one Engine, advanced by one launch per step.
  served   a queue of mixed jobs through the serving loop (admission, continuous batching,
           retirement at each job's horizon).
  cluster  decorated particles from marker particles (k-means, then the moments).
"""
import math

import numpy as np
import torch

import paper_2605_21794_amd as vp
from paper_2605_21794_amd.serve import GpuBackend, Job, Server

FIELDS = ("Q", "P", "qs", "ps", "psi")
MOMENTS = ("Mqq", "Mqp", "Mpp")


def _run(name, flow, nx, nv, ng, precision, steps, dt, **opt):
    case = {"kind": "run", "flow": flow, "nx": nx, "nv": nv, "ng": ng, "precision": precision,
            "steps": steps, "dt": dt, "elements": 1, "moments": 2, "monopole": False,
            "solver": "scan", "projection": "elem", "persistent": False}
    case.update(opt)
    return {"name": name, **case} if name else case


def _cluster(name, markers, clusters, iters, batch=0, nbatch=0):
    case = {"kind": "cluster", "markers": markers, "clusters": clusters, "iters": iters,
            "batch": batch, "nbatch": nbatch}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the linear Landau preset, the first thing a user runs: 4096 float64 particles, where
        # the step's latency and the launches are everything
        _run("landau_linear", "landau", 64, 64, 64, "fp64", 200, 0.1),
        # the default benchmark's instance with the launch shape that Engine.tune keeps for it
        _run("two_stream_tuned", "two_stream", 1024, 1024, 512, "fp32c", 300, 0.05,
             persistent=True),
        # the same flow as README's example runs it, untuned, on a lattice of odd size
        _run("two_stream_default", "two_stream", 1013, 1009, 512, "fp32c", 200, 0.05),
        # strong nonlinear Landau damping at the precision study's size: streaming many
        # particles over a small mesh
        _run("landau_nonlinear", "landau_nonlinear", 2048, 2048, 256, "fp32c", 60, 0.05),
        # P2 elements with the FFT solver on the finest mesh, float64
        _run("p2_fft", "two_stream", 512, 511, 1024, "fp64", 60, 0.05, elements=2, solver="fft"),
        # particles with second moments (k = 3)
        _run("second_moments", "two_stream", 1024, 1024, 512, "fp32c", 40, 0.05, elements=2,
             moments=3),
        # plain particle-in-cell, the paper's comparison method, at its strong Landau setting
        _run("pic", "landau_strong", 128, 1024, 128, "fp64", 100, 0.2, monopole=True),
        # a parameter sweep of uneven Landau instances in one engine
        {"name": "sweep", "kind": "sweep", "instances": 64, "steps": 50},
        # a mixed queue (Landau, two-stream, bump-on-tail) through the serving loop
        {"name": "served", "kind": "served", "jobs": 12},
        # initialisation: the particle-count study's smallest k-means, and a production one
        _cluster("kmeans_small", 40960, 4096, 10),
        _cluster("kmeans_large", 4194304, 419430, 10),
        # the mini-batch form for large marker sets
        _cluster("kmeans_minibatch", 1300001, 130000, 0, 162500, 8),
    ]


def draw(rng):
    """A case of the same ranges: sizes log-uniform, odd ones among them, every precision and
    option a job may carry."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(("run", "cluster", "sweep", "served"), (13, 5, 1, 1))[0]
    if kind == "cluster":
        m = log_int(20000, 3000000)
        k = max(64, int(m / rng.uniform(6.0, 20.0)))
        if rng.random() < 0.25:
            return _cluster(None, m, k, 0, max(k, m // rng.randint(4, 12)), rng.randint(3, 8))
        return _cluster(None, m, k, rng.randint(2, 10))
    if kind == "sweep":
        return {"kind": "sweep", "instances": rng.randint(8, 60), "steps": rng.randint(20, 50)}
    if kind == "served":
        return {"kind": "served", "jobs": rng.randint(4, 12)}
    n = log_int(1 << 12, 1 << 22)
    nx = max(48, min(2048, int(math.sqrt(n) * rng.uniform(0.6, 1.6)))) | 1
    nv = max(48, n // nx)
    opt = {}
    shape = rng.random()
    precision = rng.choices(("fp64", "fp32c", "fp32ts", "fp32"), (6, 8, 2, 1))[0]
    if shape < 0.15 and precision != "fp32":
        opt = {"elements": 2}
    elif shape < 0.25 and precision != "fp32":
        opt = {"elements": 2, "moments": 3}
    elif shape < 0.40:
        opt = {"monopole": True}
    elif shape < 0.50:
        opt = {"projection": rng.choice(("nodal", "consistent"))}
    if rng.random() < 0.2:
        opt["solver"] = "fft"
    if n <= 1 << 20 and opt.get("moments") != 3 and not opt.get("monopole") and \
            rng.random() < 0.25:
        opt["persistent"] = True
    flow = rng.choice(("landau", "two_stream", "landau_nonlinear"))
    return _run(None, flow, nx, nv, rng.choice((64, 128, 256, 512, 1024)), precision,
                max(20, min(80, (1 << 27) // (nx * nv))), 0.05, **opt)


# ---------------------------------------------------------------- inputs
def _flow(flow):
    """Domain length, velocity range and f0 = X(x) V(v) of a named flow."""
    if flow == "two_stream":
        k, alpha, vmin, vmax = 0.2, 1e-3, -8.0, 8.0
    elif flow == "bump_on_tail":
        k, alpha, vmin, vmax = 0.3, 0.04, -8.0, 10.0
    elif flow == "landau_strong":
        k, alpha, vmin, vmax = 2.0 * math.pi / 12.0, 0.5, -6.0, 6.0
    else:
        k, alpha, vmin, vmax = 0.5, (0.5 if flow == "landau_nonlinear" else 0.01), -6.0, 6.0
    return 2.0 * math.pi / k, vmin, vmax, k, alpha


def _velocity(flow, v):
    if flow == "two_stream":
        return (torch.exp(-0.5 * (v - 2.4) ** 2) + torch.exp(-0.5 * (v + 2.4) ** 2)) / \
            (2.0 * math.sqrt(2.0 * math.pi))
    if flow == "bump_on_tail":
        return (0.9 * torch.exp(-0.5 * v * v) + 0.2 * torch.exp(-2.0 * (v - 4.5) ** 2)) / \
            math.sqrt(2.0 * math.pi)
    return torch.exp(-0.5 * v * v) / math.sqrt(2.0 * math.pi)


def _lattice(flow, L, vmin, vmax, k, alpha, nx, nv, gen, moments=False, monopole=False):
    """Decorated particles of the cells of an nx x nv phase-space lattice in random order: the
    centre jittered in x, the moments by an 8-point Gauss rule (float64, on the GPU)."""
    dev = torch.device("cuda")
    t, w = (torch.from_numpy(a).to(dev) for a in np.polynomial.legendre.leggauss(8))
    dx, dv = L / nx, (vmax - vmin) / nv
    xi = torch.rand((nv, nx), generator=gen, device=dev, dtype=torch.float64) - 0.5
    perm = torch.randperm(nx * nv, generator=gen, device=dev)
    x0 = torch.arange(nx, device=dev, dtype=torch.float64) * dx
    v0 = vmin + torch.arange(nv, device=dev, dtype=torch.float64) * dv
    Q = torch.remainder(x0[None, :] + (0.5 + xi) * dx, L)
    Q = torch.where(Q >= L, torch.zeros_like(Q), Q)
    P = (v0 + 0.5 * dv)[:, None].expand(nv, nx)
    xn, vn = x0[:, None] + 0.5 * dx * (1.0 + t), v0[:, None] + 0.5 * dv * (1.0 + t)
    Xw = (1.0 + alpha * torch.cos(k * xn)) * (0.5 * dx * w)
    Vw = _velocity(flow, vn) * (0.5 * dv * w)
    X0, V0 = Xw.sum(1), Vw.sum(1)
    dvp = (v0 + 0.5 * dv)[:, None] - vn
    out = {"Q": Q, "P": P, "psi": V0[:, None] * X0[None, :]}
    if not monopole:
        th = 2.0 * math.pi / L
        c = torch.zeros_like(Q)
        c2 = torch.zeros_like(Q)
        for j in range(8):
            a = th * (Q - xn[None, :, j])
            c += Xw[None, :, j] * (torch.sin(a) / th)
            if moments:
                c2 += Xw[None, :, j] * (4.0 / th ** 2) * torch.sin(0.5 * a) ** 2
        V1, V2 = (Vw * dvp).sum(1), (Vw * dvp * dvp).sum(1)
        out["ps"] = V0[:, None] * c
        out["qs"] = -V1[:, None] * X0[None, :]
        if moments:
            out["Mqq"] = V0[:, None] * c2
            out["Mqp"] = V1[:, None] * c
            out["Mpp"] = V2[:, None] * X0[None, :]
    return {f: a.reshape(-1)[perm].contiguous() for f, a in out.items()}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _cast(state, precision):
    dt = torch.float64 if precision == "fp64" else torch.float32
    return {f: a.to(dt) for f, a in state.items()}


def _run_input(case, seed):
    L, vmin, vmax, k, alpha = _flow(case["flow"])
    st = _lattice(case["flow"], L, vmin, vmax, k, alpha, case["nx"], case["nv"], _gen(seed),
                  case["moments"] == 3, case["monopole"])
    return L, _below(_cast(st, case["precision"]), L)


def _below(state, L):
    """Positions below L also after rounding to the storage type."""
    q = state["Q"]
    state["Q"] = torch.where(q.double() >= L, torch.zeros_like(q), q)
    return state


def _sweep_instances(case, seed):
    """The sweep's recipe: alpha log-uniform in [0.01, 0.5], k uniform in [0.3, 0.6], Ng of 64,
    128 or 256, N log-uniform around [2^12, 2^16], float32 storage."""
    r = np.random.default_rng(np.random.SeedSequence([17, case["instances"]]))
    g = _gen(seed)
    out = []
    for _ in range(case["instances"]):
        alpha = math.exp(r.uniform(math.log(0.01), math.log(0.5)))
        k = r.uniform(0.3, 0.6)
        ng = int(r.choice([64, 128, 256]))
        nv = max(48, int(round(2.0 ** r.uniform(12.0, 16.0) / ng)))
        L = 2.0 * math.pi / k
        st = _lattice("landau", L, -6.0, 6.0, k, alpha, ng, nv, g)
        out.append((L, ng, 0.05, _below(_cast(st, "fp32c"), L)))
    return out


def _served_jobs(case, seed):
    """The served recipe: thirds of Landau, two-stream and bump-on-tail jobs, N log-uniform in
    [2^12, 2^20], Ng of 64 to 1024, horizons of 60 to 240 steps, all waiting at the start."""
    r = np.random.default_rng(np.random.SeedSequence([29, case["jobs"]]))
    g = _gen(seed)
    out = []
    for j in range(case["jobs"]):
        flow = ("landau", "two_stream", "bump_on_tail")[j % 3]
        L, vmin, vmax, k, alpha = _flow(flow)
        ng = int(r.choice([64, 128, 256, 512, 1024]))
        n = 2.0 ** r.uniform(12.0, 20.0)
        nx = min(ng, max(48, int(math.sqrt(n))))
        nv = max(48, int(round(n / nx)))
        st = _lattice(flow, L, vmin, vmax, k, alpha, nx, nv, g)
        out.append((L, ng, 0.025, int(r.integers(60, 241)), _below(_cast(st, "fp32c"), L)))
    return out


def _markers(case, seed):
    """Random markers of the strong Landau flow: x uniform, v Maxwellian, weights carrying the
    perturbation."""
    L, _, _, k, alpha = _flow("landau_strong")
    m, g, dev = case["markers"], _gen(seed), torch.device("cuda")
    q = torch.rand(m, generator=g, device=dev, dtype=torch.float64) * L
    p = torch.randn(m, generator=g, device=dev, dtype=torch.float64)
    w = (1.0 + alpha * torch.cos(k * q)) * (L / m)
    init = torch.randperm(m, generator=g, device=dev)[:case["clusters"]].to(torch.int32)
    bidx = None
    if case["nbatch"]:
        bidx = torch.randint(0, m, (case["nbatch"], case["batch"]), generator=g, device=dev)
        bidx = bidx.to(torch.int32)
    return L, q, p, w, init, bidx


def prepare(case, seed):
    kind = case["kind"]
    if kind == "run":
        L, st = _run_input(case, seed)
        eng = vp.Engine(case["precision"], max_slots=1)
        if case["persistent"]:
            eng.set_tuning(threads=512, ppt=8, acc_copies=4, persistent=1)
        return {"case": case, "engine": eng, "L": L, "state": st}
    if kind == "sweep":
        inst = _sweep_instances(case, seed)
        eng = vp.Engine("fp32c", max_slots=len(inst))
        return {"case": case, "engine": eng, "instances": inst}
    if kind == "served":
        srv = Server(backend=GpuBackend("fp32c", 64), budget_bytes=8 << 30, keep_state=True)
        return {"case": case, "server": srv, "jobs": _served_jobs(case, seed)}
    return {"case": case, "markers": _markers(case, seed)}


# ---------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        eng = state["engine"]
        eng.admit(0, state["state"], state["L"], case["ng"], case["dt"],
                  hist_cap=case["steps"] + 1, solver=case["solver"],
                  projection=case["projection"], monopole_only=case["monopole"],
                  element_order=case["elements"], moment_order=case["moments"])
        eng.step(case["steps"])
        h = eng.history_array(0, 0, case["steps"])
        out = dict(eng.retire(0))
        if case["monopole"]:
            out.pop("qs"), out.pop("ps")
        return {**out, "W": h["W"].copy(), "K": h["K"].copy()}
    if kind == "sweep":
        eng = state["engine"]
        for s, (L, ng, dt, st) in enumerate(state["instances"]):
            eng.admit(s, st, L, ng, dt, hist_cap=case["steps"] + 1)
        eng.step(case["steps"])
        W = np.concatenate([eng.history_array(s, 0, case["steps"])["W"]
                            for s in range(len(state["instances"]))])
        ends = [eng.retire(s) for s in range(len(state["instances"]))]
        return {**{f: torch.cat([e[f] for e in ends]) for f in FIELDS}, "W": W}
    if kind == "served":
        jobs = [Job(state=st, L=L, ng=ng, dt=dt, horizon=h)
                for L, ng, dt, h, st in state["jobs"]]
        state["server"].run(jobs)
        out = {f: torch.cat([j.final_state[f] for j in jobs]) for f in FIELDS}
        return {**out, "W": np.array([j.result["W"] for j in jobs]),
                "K": np.array([j.result["K"] for j in jobs])}
    L, q, p, w, init, bidx = state["markers"]
    out = vp.cluster_markers(q, p, w, case["clusters"], L, iters=case["iters"], init_idx=init,
                             return_assign=True, batch_idx=bidx)
    return {f: v if f == "assign" else _padded(v, case["clusters"]) for f, v in out.items()}


def _padded(v, k):
    """One entry per cluster: zeros in the place of the clusters left without members, so that
    every seed's outputs have one shape."""
    return v if v.numel() == k else torch.nn.functional.pad(v, (0, k - v.numel()))


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes: every input read once and every output written once.  Operations: the float64
    arithmetic of one update (about 35 for a P1 particle, 25 without dipoles, 50 with P2
    elements, 95 with second moments), and for the k-means about ten centres of five
    operations each per marker and pass."""
    kind = case["kind"]
    if kind == "run":
        n, el = case["nx"] * case["nv"], 8 if case["precision"] == "fp64" else 4
        arrays = 5 if case["monopole"] else 15 if case["moments"] == 3 else 9
        per = 95 if case["moments"] == 3 else 50 if case["elements"] == 2 else \
            25 if case["monopole"] else 35
        return {"bytes": float(arrays * el * n + 96 * case["steps"]),
                "flops": float(per * n * case["steps"])}
    if kind == "sweep":
        r = np.random.default_rng(np.random.SeedSequence([17, case["instances"]]))
        n = 0
        for _ in range(case["instances"]):
            r.uniform(), r.uniform()
            ng = int(r.choice([64, 128, 256]))
            n += ng * max(48, int(round(2.0 ** r.uniform(12.0, 16.0) / ng)))
        return {"bytes": 36.0 * n + 96.0 * case["steps"] * case["instances"],
                "flops": 35.0 * n * case["steps"]}
    if kind == "served":
        r = np.random.default_rng(np.random.SeedSequence([29, case["jobs"]]))
        b = f = 0.0
        for _ in range(case["jobs"]):
            ng = int(r.choice([64, 128, 256, 512, 1024]))
            n = 2.0 ** r.uniform(12.0, 20.0)
            nx = min(ng, max(48, int(math.sqrt(n))))
            n = nx * max(48, int(round(n / nx)))
            b += 36.0 * n
            f += 35.0 * n * int(r.integers(60, 241))
        return {"bytes": b, "flops": f}
    m, k = case["markers"], case["clusters"]
    passes = case["iters"] + 1
    seen = m * passes + case["batch"] * case["nbatch"]
    return {"bytes": 28.0 * m + 44.0 * k + 4.0 * case["batch"] * case["nbatch"],
            "flops": 50.0 * seen + 10.0 * seen}


# ---------------------------------------------------------------- the same in plain float64
def _p1_load(Q, psi, ps, ng, inv_h):
    x = Q * inv_h
    i = torch.clamp(torch.floor(x), 0, ng - 1)
    s = torch.clamp(x - i, 0.0, 1.0)
    i = i.long()
    b = torch.zeros(ng, dtype=torch.float64, device=Q.device)
    b.index_add_(0, i, psi * (1.0 - s) + ps * inv_h)
    b.index_add_(0, (i + 1) % ng, psi * s - ps * inv_h)
    return b


def _p2_load(Q, psi, ps, ng, inv_h, Mqq):
    x = Q * inv_h
    i = torch.clamp(torch.floor(x), 0, ng - 1)
    s = torch.clamp(x - i, 0.0, 1.0)
    i = i.long()
    m = 0.0 if Mqq is None else 0.5 * Mqq * inv_h ** 2
    b = torch.zeros(2 * ng, dtype=torch.float64, device=Q.device)
    b.index_add_(0, i, psi * (1 - s) * (1 - 2 * s) - ps * (4 * s - 3) * inv_h + 4 * m)
    b.index_add_(0, ng + i, psi * 4 * s * (1 - s) - ps * (4 - 8 * s) * inv_h - 8 * m)
    b.index_add_(0, (i + 1) % ng, psi * s * (2 * s - 1) - ps * (4 * s - 1) * inv_h + 4 * m)
    return b


def _gauss(b):
    """E_e with E_e - E_{e-1} = b_e and sum E = 0."""
    E = torch.cumsum(b, 0)
    return E - E.mean()


def _consistent(bt, h):
    """g with (h/6)(g_{j-1} + 4 g_j + g_{j+1}) = -b~_j, by its Fourier symbol."""
    ng = bt.numel()
    th = 2.0 * math.pi * torch.arange(ng // 2 + 1, device=bt.device, dtype=torch.float64) / ng
    return torch.fft.irfft(-torch.fft.rfft(bt) / ((h / 6.0) * (4.0 + 2.0 * torch.cos(th))), ng)


def _simulate(st, L, ng, dt, steps, elements=1, moments=2, projection="elem"):
    """The kick-drift-kick cycle in plain float64; returns the final state and the W and K of
    every integer step before it, and of the last one."""
    Q, P, psi = (st[f].double() for f in ("Q", "P", "psi"))
    qs = st["qs"].double() if "qs" in st else torch.zeros_like(Q)
    ps = st["ps"].double() if "ps" in st else torch.zeros_like(Q)
    Mqq, Mqp, Mpp = (st[f].double() for f in MOMENTS) if moments == 3 else (None,) * 3
    inv_h, h = ng / L, L / ng
    dip = "ps" in st

    def field():
        if elements == 1:
            b = _p1_load(Q, psi, ps, ng, inv_h)
            bt = b - b.mean()
            E = _gauss(bt)
            W = 0.5 * h * (E * E).sum()
            if projection == "elem":
                g = -(bt + torch.roll(bt, -1)) / (2.0 * h)
            else:
                g = -bt / h if projection == "nodal" else _consistent(bt, h)
        else:
            b = _p2_load(Q, psi, ps, ng, inv_h, Mqq)
            mean = b.sum() / ng
            bm = b[ng:] - (2.0 / 3.0) * mean
            bv = b[:ng] + 0.5 * (b[ng:] + torch.roll(b[ng:], 1)) - mean
            E = _gauss(bv)
            W = 0.5 * h * (E * E).sum() + (3.0 * h / 32.0) * (bm * bm).sum()
            g = -3.0 * bm / (2.0 * h)
        x = Q * inv_h
        i = torch.clamp(torch.floor(x), 0, ng - 1)
        s = torch.clamp(x - i, 0.0, 1.0)
        i = i.long()
        if elements == 2:
            return E[i] - h * g[i] * (s - 0.5), g[i], W
        if projection == "elem":
            return E[i], g[i], W
        return E[i], (1.0 - s) * g[i] + s * g[(i + 1) % ng], W

    Ws, Ks = [], []
    half = 0.5 * dt
    Ea, ga, W = field()

    def kick():
        nonlocal P, qs, Mqp, Mpp
        P = P + half * Ea
        if dip:
            qs = qs + half * ps * ga
        if moments == 3:
            Mpp = Mpp - 2.0 * half * ga * Mqp + (half * ga) ** 2 * Mqq
            Mqp = Mqp - half * ga * Mqq

    def kinetic():
        K = (0.5 * psi * P * P + qs * P).sum()
        return K + 0.5 * Mpp.sum() if moments == 3 else K

    for _ in range(steps):
        Ws.append(W)
        Ks.append(kinetic())
        kick()
        Q = Q + dt * P
        Q = torch.where(Q < 0.0, Q + L, Q)
        Q = torch.where(Q >= L, Q - L, Q)
        if dip:
            ps = ps - dt * qs
        if moments == 3:
            Mqq = Mqq + 2.0 * dt * Mqp + dt * dt * Mpp
            Mqp = Mqp + dt * Mpp
        Ea, ga, W = field()
        kick()
    out = {"Q": Q, "P": P, "qs": qs, "ps": ps, "psi": psi}
    if moments == 3:
        out.update(Mqq=Mqq, Mqp=Mqp, Mpp=Mpp)
    return out, torch.stack(Ws + [W]), torch.stack(Ks + [kinetic()])


def _kmeans(case, L, q, p, w, init):
    """Lloyd's iterations by full distance rows, then the decorated particles."""
    k, m = case["clusters"], q.numel()
    cq, cp = q[init.long()].clone(), p[init.long()].clone()
    rows = max(1, (1 << 26) // k)
    for it in range(case["iters"] + 1):
        a = torch.empty(m, dtype=torch.int64, device=q.device)
        for r in range(0, m, rows):
            d2 = (q[r:r + rows, None] - cq[None, :]) ** 2 + (p[r:r + rows, None] - cp[None, :]) ** 2
            a[r:r + rows] = torch.argmin(d2, dim=1)
        sums = [torch.zeros(k, dtype=torch.float64, device=q.device).index_add_(0, a, v)
                for v in (w, w * q, w * p)]
        some = sums[0] > 0.0
        zq, zp = sums[1] / sums[0], sums[2] / sums[0]
        if it < case["iters"]:
            cq, cp = torch.where(some, zq, cq), torch.where(some, zp, cp)
    d2 = (q - zq[a]) ** 2 + (p - zp[a]) ** 2
    near = torch.full((k,), math.inf, dtype=torch.float64, device=q.device)
    near.scatter_reduce_(0, a, d2, "amin")
    at = torch.arange(m, device=q.device)
    first = torch.full((k,), m, dtype=torch.int64, device=q.device)
    first.scatter_reduce_(0, a, torch.where(d2 == near[a], at, torch.full_like(at, m)), "amin")
    c = torch.where(some, first, torch.zeros_like(first))
    ps = torch.zeros(k, dtype=torch.float64, device=q.device).index_add_(
        0, a, w * (L / (2.0 * math.pi)) * torch.sin(2.0 * math.pi * (q[c][a] - q) / L))
    qs = torch.zeros(k, dtype=torch.float64, device=q.device).index_add_(0, a, -w * (p[c][a] - p))
    out = {"Q": q[c], "P": p[c], "qs": qs, "ps": ps, "psi": sums[0]}
    return {**{f: _padded(v[some], k) for f, v in out.items()}, "assign": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "run":
        L, st = _run_input(case, seed)
        out, W, K = _simulate(st, L, case["ng"], case["dt"], case["steps"], case["elements"],
                              case["moments"], case["projection"])
        if case["monopole"]:
            out.pop("qs"), out.pop("ps")
        return {**out, "W": W[:-1], "K": K[:-1]}
    if kind == "sweep":
        ends = [_simulate(st, L, ng, dt, case["steps"])
                for L, ng, dt, st in _sweep_instances(case, seed)]
        return {**{f: torch.cat([e[0][f] for e in ends]) for f in FIELDS},
                "W": torch.cat([e[1][:-1] for e in ends])}
    if kind == "served":
        ends = [_simulate(st, L, ng, dt, h) for L, ng, dt, h, st in _served_jobs(case, seed)]
        return {**{f: torch.cat([e[0][f] for e in ends]) for f in FIELDS},
                "W": torch.stack([e[1][-1] for e in ends]),
                "K": torch.stack([e[2][-1] for e in ends])}
    if case["nbatch"] or case["markers"] * case["clusters"] * (case["iters"] + 1) > 1 << 37:
        return None
    L, q, p, w, init, _ = _markers(case, seed)
    return _kmeans(case, L, q, p, w, init)
