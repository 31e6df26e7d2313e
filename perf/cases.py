"""Workloads of the library as its users run them, through the public entry points.

Each case is one way a program uses the package: plans replayed on a model (the
solver's inner loop), a batch of clouds in one graph, the one-call path on a list of
origins, bare ray lists, adaptive direction sets, and the learned closure's inference
and training.  Sizes follow bench.py and the tests: the 1 200-point sphere, the
50 000-point wind and octree-like grid, SPH-like clouds, F = 31, 64 and 2 x 48.

Meshes are made on the GPU from a seed: `cloud` is a ball of irregular points, denser
towards the centre, whose neighbours are the points within 1.55 mean spacings before
the radial stretching (about 14 each, as many as a Delaunay point has); `grid` is a
graded rectilinear grid with its 26 touching cells (the octree's leaves), cells in
memory order.  Cloud points are numbered at random, as generated particles are.
"""
import math

import torch

import paper_2011_14998_amd as rt

DEV = "cuda"


# ------------------------------------------------------------------ cases

def listed():
    plan = dict(kind="plan", mesh="cloud", P=50000, nside=2, blocks=1, nf=64, f64=False, moving=True,
                schedule="spatial", dtau=0.0, dv=0.0, hermite=False)
    return [
        # the smallest replay a solver iterates on: static, FP64, launches and latency count
        dict(plan, name="sphere plan f64", P=1200, nside=1, nf=31, f64=True, moving=False),
        # the analytic wind at the resolution of the benchmark
        dict(plan, name="wind plan f32", nside=4),
        # the same path in FP64, a ragged size
        dict(plan, name="wind plan f64", P=20011, f64=True),
        # two lines of 48 frequencies on octree-like cells
        dict(plan, name="grid plan 2x48", mesh="grid", nside=4, blocks=2, nf=48),
        # lines refined by velocity sampling (a third of a Doppler width)
        dict(plan, name="wind velocity-sampled", P=10007, dv=1.0 / 3.0),
        # lines refined by optical depth under the fourth-order rows (FP64: their weights are ill-conditioned)
        dict(plan, name="wind fourth-order f64", P=10007, f64=True, dtau=1.0, hermite=True),
        # clouds of many sizes solved together
        dict(kind="batch", name="16 clouds", n=16, P_lo=4000, P_hi=40000, nside=2, blocks=1, nf=64, f64=False),
        # one call on a list of origins: what re-solves a part of a model at high angular resolution
        dict(kind="compute", name="subset at nside 8", mesh="cloud", P=100000, n=3001, nside=8, blocks=1, nf=64,
             f64=False, moving=True),
        # ray lists alone, for a caller's own solver
        dict(kind="trace", name="ray lists", mesh="cloud", P=100000, n=20011, nside=2),
        # directions refined towards the points seen from each origin, then the solve over them
        dict(kind="adaptive", name="adaptive directions", mesh="grid", P=50000, n=1000, lmin=1, lmax=4, sample=10000,
             blocks=2, nf=48),
        # the closure's inference on one chunk of points
        dict(kind="infer", name="closure inference", P=65536, nf=64),
        # the closure's training steps
        dict(kind="train", name="closure training", N=1 << 20, batch=8192, steps=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plan", "plan", "plan", "plan", "batch", "compute", "compute", "trace", "adaptive", "infer",
                       "train"])
    blocks = rng.choice([1, 1, 1, 2, 2, 3])
    nf = rng.randint(16, 64 if blocks == 1 else 48 if blocks == 2 else 32)
    mesh = rng.choice(["cloud", "cloud", "grid"])
    f64 = rng.random() < 0.3
    if kind == "plan":
        refine = rng.choice(["no", "no", "no", "no", "dv", "dtau", "hermite"])
        P = _log(rng, 1000, 50000 if refine == "no" else 10000)
        nside = rng.choice([n for n in (1, 2, 4) if P * n * n <= (400000 if refine == "no" else 40000)])
        return dict(kind=kind, mesh="cloud" if refine != "no" else mesh, P=P, nside=nside, blocks=blocks, nf=nf,
                    f64=True if refine == "hermite" else f64, moving=refine != "no" or rng.random() < 0.8,
                    schedule=rng.choice(["spatial", "spatial", "spatial", "binned", "direct"]),
                    dtau=rng.uniform(0.5, 2.0) if refine in ("dtau", "hermite") else 0.0,
                    dv=rng.uniform(0.3, 1.0) if refine == "dv" else 0.0, hermite=refine == "hermite")
    if kind == "batch":
        lo = _log(rng, 500, 4000)
        return dict(kind=kind, n=rng.randint(2, 16), P_lo=lo, P_hi=lo * rng.randint(2, 8), nside=rng.choice([1, 2]),
                    blocks=blocks, nf=nf, f64=f64)
    if kind == "compute":
        P = _log(rng, 2000, 100000)
        nside = rng.choice([1, 2, 4, 8])
        return dict(kind=kind, mesh=mesh, P=P, n=min(P, _log(rng, 50, 190000 // (nside * nside))), nside=nside,
                    blocks=blocks, nf=nf, f64=f64, moving=rng.random() < 0.8)
    if kind == "trace":
        P = _log(rng, 2000, 100000)
        return dict(kind=kind, mesh=mesh, P=P, n=min(P, _log(rng, 100, 20000)), nside=rng.choice([1, 2]))
    if kind == "adaptive":
        P = _log(rng, 5000, 50000)
        lmin = rng.choice([0, 1])
        return dict(kind=kind, mesh="grid" if mesh == "grid" else "cloud", P=P, n=_log(rng, 50, 1000), lmin=lmin,
                    lmax=lmin + rng.choice([2, 3]), sample=_log(rng, 1000, 10000) if P > 10000 else 1000,
                    blocks=blocks, nf=nf)
    if kind == "infer":
        return dict(kind=kind, P=_log(rng, 500, 65536), nf=rng.randint(16, 64))
    return dict(kind="train", N=_log(rng, 20000, 1 << 20), batch=_log(rng, 500, 8192), steps=rng.randint(2, 16))


# ------------------------------------------------------------------ models

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _csr(P, a, b):
    """Rows of ascending neighbour ids from directed edges a -> b (both directions present)."""
    key = torch.sort(a * P + b).values
    off = torch.zeros(P + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(key // P, minlength=P), 0)
    return off, (key % P).to(torch.int32)


def _offsets(k):
    r = torch.arange(-k, k + 1, device=DEV)
    o = torch.stack(torch.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    return o[(o != 0).any(1)]


def _cloud(P, g):
    """P points of a ball: one per cell of a cubic grid, the P nearest to its centre kept, then
    stretched so that the spacing grows e^3 from the centre to the edge; ids at random."""
    n = int(math.ceil((P * 6.0 / math.pi) ** (1.0 / 3.0))) + 2
    c = torch.stack(torch.meshgrid(*[torch.arange(n, device=DEV)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = c + torch.rand(c.shape, generator=g, device=DEV, dtype=torch.float64)
    r = (x - 0.5 * n).norm(dim=1)
    sel = torch.topk(r, P, largest=False).indices
    num = torch.full((n, n, n), -1, dtype=torch.int64, device=DEV)
    num.view(-1)[sel] = torch.randperm(P, generator=g, device=DEV)
    src, dst = [], []
    cs, xs, ns = c[sel], x[sel], num.view(-1)[sel]
    xg = x.reshape(n, n, n, 3)
    for o in _offsets(2):
        q = cs + o
        ok = ((q >= 0) & (q < n)).all(1)
        q = q.clamp(0, n - 1)
        k = num[q[:, 0], q[:, 1], q[:, 2]]
        ok &= (k >= 0) & ((xg[q[:, 0], q[:, 1], q[:, 2]] - xs).square().sum(1) < 1.55 * 1.55)
        src.append(ns[ok])
        dst.append(k[ok])
    off, idx = _csr(P, torch.cat(src), torch.cat(dst))
    d = (xs - 0.5 * n) / r[sel].max()
    rr = d.norm(dim=1, keepdim=True).clamp_min(1e-12)
    pos = torch.empty(P, 3, dtype=torch.float64, device=DEV)
    pos[ns] = d / rr * torch.expm1(3.0 * rr) / math.expm1(3.0)
    return pos.contiguous(), off, idx


def _grid_dims(P):
    a = max(2, int(round(P ** (1.0 / 3.0))))
    return a, a, max(2, P // (a * a))


def _grid(P, g):
    """A rectilinear grid with graded spacings, cells in memory order, 26 touching neighbours; a
    point lies within a fiftieth of a cell of the cell's centre (no ray is decided by rounding)."""
    dims = _grid_dims(P)
    ax = []
    for n in dims:
        t = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
        ph = torch.rand(3, generator=g, device=DEV, dtype=torch.float64)
        ax.append(t + 0.08 * torch.sin(2 * math.pi * (t + ph[0])) + 0.03 * torch.sin(4 * math.pi * (t + ph[1])))
    pos = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    pos += (torch.rand(pos.shape, generator=g, device=DEV, dtype=torch.float64) - 0.5) * (0.04 / max(dims))
    n0, n1, n2 = dims
    c = torch.stack(torch.meshgrid(*[torch.arange(n, device=DEV) for n in dims], indexing="ij"), -1).reshape(-1, 3)
    lin = torch.arange(n0 * n1 * n2, device=DEV)
    top = torch.tensor(dims, device=DEV)
    src, dst = [], []
    for o in _offsets(1):
        q = c + o
        ok = ((q >= 0) & (q < top)).all(1)
        q = q[ok]
        src.append(lin[ok])
        dst.append((q[:, 0] * n1 + q[:, 1]) * n2 + q[:, 2])
    off, idx = _csr(len(lin), torch.cat(src), torch.cat(dst))
    return pos.contiguous(), off, idx


def _modes(pos, g, k_max=4.0):
    """A smooth random field of unit variance on the unit box."""
    f = torch.zeros(len(pos), dtype=torch.float64, device=DEV)
    for _ in range(8):
        k = torch.rand(3, generator=g, device=DEV, dtype=torch.float64) * 2 * k_max - k_max
        ph = torch.rand(1, generator=g, device=DEV, dtype=torch.float64)
        f += 0.5 * torch.sin(2 * math.pi * (pos @ k + ph))
    return f


def _grid_x(blocks, nf):
    dx = 10.0 / (nf - 1)
    return [nf] * blocks, [dx] * blocks, [-5.0] * blocks


def _physics(mesh, pos, g, blocks, nf, f64, moving, flow="wind"):
    """Opacity, emissivity, velocity (Doppler widths) and boundary intensity on the points."""
    dt = torch.float64 if f64 else torch.float32
    x = -5.0 + 10.0 / (nf - 1) * torch.arange(nf, device=DEV, dtype=torch.float64)
    prof = torch.cat([torch.exp(-x * x) / (b + 1) for b in range(blocks)])
    if mesh == "grid":  # log-normal density, random flow of 3 Doppler widths
        rho = torch.exp(_modes(pos, g) - 0.5)
        chi0, S = 100.0, rho ** 0.3
        vel = torch.stack([3.0 / math.sqrt(3.0) * _modes(pos, g) for _ in range(3)], 1)
    else:
        r = 100.0 * pos.norm(dim=1)
        amp = torch.exp(0.1 * _modes(pos, g))
        if flow == "wind":  # rho ~ r^-2, accelerating radially to 20 Doppler widths
            rho = 100.0 * amp / (1.0 + r * r)
            chi0, S = 10.0, 1.0 / (1.0 + r)
            vel = pos / pos.norm(dim=1, keepdim=True).clamp_min(1e-12) * (20.0 * torch.sqrt(r / (1.0 + r)))[:, None]
        else:  # a rotating Plummer-like sphere
            rho = 100.0 * amp * (1.0 + (0.1 * r) ** 2) ** -2.5
            chi0, S = 1.0, rho ** 0.3
            R = pos[:, :2].norm(dim=1).clamp_min(0.01)
            v = 10.0 * torch.sqrt(0.1 / R)
            vel = torch.stack([-v * pos[:, 1] / R, v * pos[:, 0] / R, torch.zeros_like(v)], 1)
    chi = (chi0 * rho[:, None] * (prof[None, :] + 1e-4)).to(dt).contiguous()
    eta = (chi.double() * S[:, None]).to(dt).contiguous()
    I_bc = torch.full((blocks * nf,), 0.01, dtype=torch.float64, device=DEV)
    return chi, eta, vel.float().contiguous() if moving else None, I_bc


def _model(c, g, P=None, flow="wind"):
    mesh = c.get("mesh", "cloud")
    pos, off, idx = (_grid if mesh == "grid" else _cloud)(P or c["P"], g)
    if mesh == "cloud":
        pos = pos * 100.0
    chi, eta, vel, I_bc = _physics(mesh, pos / 100.0 if mesh == "cloud" else pos, g, c.get("blocks", 1),
                                   c.get("nf", 64), c.get("f64", False), c.get("moving", True), flow)
    return dict(pos=pos, off=off, idx=idx, vel=vel, chi=chi, eta=eta, I_bc=I_bc)


def _handle(m):
    return rt.Model(m["pos"], m["off"], m["idx"], m["vel"])


def _batch_sizes(c):
    return [int(round(c["P_lo"] * (c["P_hi"] / c["P_lo"]) ** (k / max(1, c["n"] - 1)))) for k in range(c["n"])]


def _weights(g):
    """Network parameters: N(0, 2/fan_in) (the head 1/fan_in), biases 0."""
    w = [torch.randn(a, 256, generator=g, device=DEV) * math.sqrt(2.0 / f) for a, f in ((16, 12), (256, 256), (256, 256))]
    head = torch.randn(256, 2, generator=g, device=DEV) / 16.0
    zero = torch.zeros(256, device=DEV)
    return torch.cat([t.reshape(-1) for t in (w[0], zero, w[1], zero, w[2], zero, head, zero[:2])])


def _origins(P, n, g):
    return torch.randperm(P, generator=g, device=DEV)[:n].to(torch.int32).contiguous()


def _inputs(case, seed):
    """The plain tensors of a case, from the seed alone."""
    g = _gen(seed)
    c = case
    if c["kind"] == "batch":
        return [_model(c, g, P=P, flow="disc") for P in _batch_sizes(c)]
    if c["kind"] == "infer":
        m = _model(dict(c, moving=False), g)
        n, F, R = c["P"], c["nf"], 6
        S = (m["eta"] / m["chi"]).double()
        u = S[:, None, :] * torch.exp(0.5 * torch.randn(n, R, F, generator=g, device=DEV, dtype=torch.float64))
        m["u"] = u.float().contiguous()
        m["J1"] = u.mean(1).float().contiguous()
        m["w"] = _weights(g)
        m["fx"] = (-5.0 + 10.0 / (F - 1) * torch.arange(F, device=DEV, dtype=torch.float64)).float()
        m["mean"] = [-3.0, -4.0, -3.0, -4.0, -3.0, 0.5, 0.3, 0.1, 1.0, -3.0, 0.0, 2.6, 0.7, -0.9, 0.5, 0.0]
        m["istd"] = [0.5, 0.3, 0.5, 0.3, 0.5, 2.0, 4.0, 9.0, 1.0, 0.3, 1.7, 5.0, 3.0, 3.0, 6.0, 0.0]
        return m
    if c["kind"] == "train":
        X = torch.randn(c["N"], 16, generator=g, device=DEV)
        X[:, 15] = 0.0
        T = 0.3 * torch.tanh(X[:, 0] - X[:, 3]) + 0.1 * X[:, 7] * X[:, 9] + 0.05 * torch.randn(
            c["N"], generator=g, device=DEV)
        return dict(X=X.to(torch.bfloat16).view(torch.int16).contiguous(), T=T.contiguous(), w=_weights(g))
    m = _model(c, g)
    P = len(m["pos"])
    if c["kind"] in ("compute", "trace", "adaptive"):
        m["origins"] = _origins(P, min(P, c["n"]), g)
    if c["kind"] == "adaptive":
        m["sample"] = _origins(P, min(P, c["sample"]), g)
    return m


SCHED = {"spatial": rt.SCHED_SPATIAL, "binned": rt.SCHED_BINNED, "direct": rt.SCHED_DIRECT}


def prepare(case, seed):
    c, m = case, _inputs(case, seed)
    s = dict(case=c, m=m)
    if c["kind"] in ("train", "infer"):
        s["net"] = rt.MLP()
        s["net"].set_params(m["w"].cpu().numpy())
    if c["kind"] == "train":
        return s
    if c["kind"] == "infer":
        s["model"] = _handle(m)
        n = c["P"] * c["nf"]
        s["feat"] = torch.empty(n, 16, device=DEV)
        s["X"] = torch.empty(n, 16, dtype=torch.int16, device=DEV)
        s["Y"] = torch.empty(n, 2, device=DEV)
        s["J"] = torch.empty(c["P"], c["nf"], device=DEV)
        return s
    if c["kind"] == "trace":
        s["model"], s["set"] = _handle(m), rt.DirSet.uniform(c["nside"])
        return s
    prec = rt.RT_F64 if c.get("f64") else rt.RT_F32
    ln, dx, _ = _grid_x(c["blocks"], c["nf"])
    if c["kind"] == "batch":
        s["set"] = rt.DirSet.uniform(c["nside"])
        s["J"] = [torch.empty_like(x["chi"]) for x in m]
        s["batch"] = rt.Batch([_handle(x) for x in m], s["set"], [x["chi"] for x in m], [x["eta"] for x in m], ln, dx,
                              m[0]["I_bc"], s["J"], precision=prec, schedule=rt.SCHED_SPATIAL)
        return s
    s["model"] = _handle(m)
    if c["kind"] == "plan":
        s["set"] = rt.DirSet.uniform(c["nside"])
        s["J"] = torch.empty_like(m["chi"])
        s["plan"] = rt.Plan(s["model"], s["set"], m["chi"], m["eta"], ln, dx, m["I_bc"], s["J"], precision=prec,
                            schedule=SCHED[c["schedule"]], dtau_max=c["dtau"], dv_max=c["dv"],
                            scheme=rt.SCHEME_HERMITE if c["hermite"] else rt.SCHEME_FEAUTRIER2)
        return s
    n, F = m["origins"].numel(), c["blocks"] * c["nf"]
    s["J"] = torch.empty(n, F, dtype=m["chi"].dtype, device=DEV)
    if c["kind"] == "compute":
        s["set"] = rt.DirSet.uniform(c["nside"])
        pairs = s["set"].R
    else:
        pairs = 6 * 4 ** c["lmin"] * ((2 ** (c["lmax"] - c["lmin"]) - 1) // 2 + 2 ** (c["lmax"] - c["lmin"]) + 1)
    # the workspace a program keeps between calls: every origin in one chunk at 96 entries a ray
    per = rt.compute_J_workspace(rt.DirSet.uniform(8), 64, F, precision=prec, mean_entries=96.0) / (64.0 * 384.0)
    s["ws"] = torch.empty(int(1.2 * per * n * pairs) + (64 << 20), dtype=torch.uint8, device=DEV)
    return s


def run(state):
    c, m = state["case"], state["m"]
    kind = c["kind"]
    if kind == "plan":
        state["plan"].run()
        return state["J"]
    if kind == "batch":
        state["batch"].run()
        return state["J"]
    if kind == "trace":
        cap = int(2 * state["set"].R * m["origins"].numel() * _mean_ray(c["mesh"], c["P"], 1.2))
        off, ids, Z, total = rt.trace_once(state["model"], state["set"], cap, origins=m["origins"])
        ids[total:].fill_(-1)  # the rest of the lists' space holds no entries
        Z[total:].fill_(0.0)
        return dict(off=off, ids=ids, Z=Z, total=total)
    if kind == "train":
        state["net"].train(m["X"], m["T"], n_steps=c["steps"], batch=c["batch"], total_steps=20000, lr=2e-3,
                           lr_final=1e-5, seed=7)
        return state["net"].get_params()
    if kind == "infer":
        feat = rt.closure_features(state["model"], m["chi"], m["eta"], m["fx"], m["J1"], u=m["u"], feat=state["feat"])
        X = rt.closure_normalize(feat, m["mean"], m["istd"], X=state["X"])
        Y = state["net"].forward(X, Y=state["Y"])
        J, _, _ = rt.closure_apply(m["J1"], Y, math.inf, J=state["J"])
        return dict(X=X, Y=Y, J=J)
    ln, dx, _ = _grid_x(c["blocks"], c["nf"])
    prec = rt.RT_F64 if c.get("f64") else rt.RT_F32
    ds = state["set"] if kind == "compute" else rt.DirSet.adaptive(state["model"], c["lmin"], c["lmax"], m["sample"],
                                                                   origins=m["origins"])
    return rt.compute_J(state["model"], ds, m["chi"], m["eta"], ln, dx, m["I_bc"], origins=m["origins"],
                        J=state["J"], ws=state["ws"], precision=prec)


# ------------------------------------------------------------------ work

def _mean_ray(mesh, P, margin=1.0):
    """List entries of a ray: measured 0.71-0.81 P^(1/3) on clouds, 1.0-1.38 on grids."""
    return margin * (1.25 if mesh == "grid" else 0.75) * P ** (1.0 / 3.0)


def _path_work(mesh, P, n, pairs, F, es, moving, refine=1.0):
    """Walk and sweep of n origins: each table once; per walk step the row's candidates, 24 operations
    each, and per line point and frequency about 22 (interpolation, optical depth, one row)."""
    deg = 26 if mesh == "grid" else 14
    steps = n * 2.0 * pairs * _mean_ray(mesh, P)
    nbytes = P * (24 + 8 + 12 * moving + 4 * deg + 2 * es * F) + es * n * F
    return nbytes, steps * (24.0 * deg + refine * 22.0 * F)


def work(case):
    c = case
    if c["kind"] == "train":
        one = 2.0 * (16 * 256 + 2 * 256 * 256 + 2 * 256)
        return dict(bytes=c["steps"] * (c["batch"] * 36.0 + 136450 * 28.0), flops=3.0 * c["steps"] * c["batch"] * one)
    if c["kind"] == "infer":
        n = c["P"] * c["nf"]
        return dict(bytes=n * (8.0 + 4 + 24 + 32 + 8 + 4) + c["P"] * 90.0,
                    flops=n * 2.0 * (16 * 256 + 2 * 256 * 256 + 2 * 256))
    if c["kind"] == "trace":
        _, fl = _path_work(c["mesh"], c["P"], c["n"], 6 * c["nside"] ** 2, 0, 0, 0)
        rays = c["n"] * 12.0 * c["nside"] ** 2
        return dict(bytes=c["P"] * 88.0 + rays * (8 + 12 * _mean_ray(c["mesh"], c["P"])), flops=fl)
    es = 8 if c.get("f64") else 4
    F = c["blocks"] * c["nf"]
    if c["kind"] == "batch":
        b = [_path_work("cloud", P, P, 6 * c["nside"] ** 2, F, es, 1) for P in _batch_sizes(c)]
        return dict(bytes=sum(x[0] for x in b), flops=sum(x[1] for x in b))
    if c["kind"] == "adaptive":
        k = c["lmax"] - c["lmin"]
        nb, fl = _path_work(c["mesh"], c["P"], c["n"], 6 * 4 ** c["lmin"] * ((2 ** k - 1) / 2 + 2 ** k), F, es, 1)
        return dict(bytes=nb, flops=fl + c["n"] * c["sample"] * 60.0)
    refine = 4.0 if c.get("dv") else 2.0 if c.get("dtau") else 1.0
    nb, fl = _path_work(c["mesh"], c["P"], c.get("n", c["P"]), 6 * c["nside"] ** 2, F, es, int(c["moving"]), refine)
    return dict(bytes=nb, flops=fl)


# ------------------------------------------------------------------ the results in 64 bits

def _directions(nside):
    """Centres of one pixel of every antipodal pair of the ring-scheme HEALPix pixels, ascending:
    a pixel is kept when it lies on the upper half sphere, or on the equator's first half turn."""
    out = []
    for i in range(1, 2 * nside + 1):
        if i < nside:
            z, n, s = 1.0 - i * i / (3.0 * nside * nside), 4 * i, 0.5
        else:
            z, n, s = 4.0 / 3.0 - 2.0 * i / (3.0 * nside), 4 * nside, 0.5 * ((i - nside + 1) % 2)
        for j in range(n if i < 2 * nside else n // 2):
            phi = 2.0 * math.pi * (j + s) / n
            st = math.sqrt(max(0.0, 1.0 - z * z))
            out.append((st * math.cos(phi), st * math.sin(phi), z))
    return out


def _padded(m):
    deg = m["off"][1:] - m["off"][:-1]
    P, D = len(deg), int(deg.max())
    nbr = torch.full((P, D), -1, dtype=torch.int64, device=DEV)
    row = torch.repeat_interleave(torch.arange(P, device=DEV), deg)
    nbr[row, torch.arange(len(row), device=DEV) - m["off"][row]] = m["idx"].long()
    return nbr


def _walk(m, nbr, org, d):
    """Lists of one direction from every origin: step s holds (rays, points, projections)."""
    pos = m["pos"]
    cur, Zc = org.clone(), torch.zeros(len(org), dtype=torch.float64, device=DEV)
    live = torch.arange(len(org), device=DEV)
    steps = []
    while len(live):
        k = nbr[cur]
        R = pos[k.clamp_min(0)] - pos[org[live]][:, None, :]
        Z = R @ d
        D = (R - Z[..., None] * d).square().sum(-1)
        D = torch.where((k >= 0) & (Z > Zc[:, None]), D, math.inf)
        best, j = D.min(1)
        ok = torch.isfinite(best)
        live, cur, Zc = live[ok], k[ok, j[ok]], Z[ok, j[ok]]
        if len(live):
            steps.append((live, cur, Zc))
    return steps


def _optics(m, q, shift, ln, dx):
    """chi, eta of points q read at f - shift/dx in each block, clamped at its ends."""
    chi, eta, F0, c, e = m["chi"], m["eta"], 0, [], []
    for n, w in zip(ln, dx):
        if shift is None:
            c.append(chi[q, F0:F0 + n].double())
            e.append(eta[q, F0:F0 + n].double())
        else:
            s = shift / w
            k = torch.floor(s)
            t = (s - k)[:, None]
            f = torch.arange(n, device=DEV)[None, :] - k.long()[:, None]
            a, b = F0 + f.clamp(0, n - 1), F0 + (f - 1).clamp(0, n - 1)
            for tab, out in ((chi, c), (eta, e)):
                rows = tab[q].double()
                out.append((1 - t) * rows.gather(1, a) + t * rows.gather(1, b))
        F0 += n
    return torch.cat(c, 1), torch.cat(e, 1)


def _side(m, steps, org, d, sign, co, I, ln, dx):
    """One side of the lines eliminated from the far end: (step to the origin, pivot, right-hand side)."""
    n, F = len(org), m["chi"].shape[1]
    z = lambda v: torch.full((n, F), v, dtype=torch.float64, device=DEV)  # noqa: E731
    g, y, a, c1, S1 = z(1.0), I.expand(n, F).clone(), z(0.0), z(0.0), z(0.0)
    vel = None if m["vel"] is None else m["vel"].double()

    def row(r, cn, ds):  # the row of the point whose values are held, its inner step towards opacity cn
        b = 0.5 * (c1[r] + cn) * ds[:, None]
        h = 0.5 * (a[r] + b)
        G = g[r] + h  # g: the pivot the outer row passes on
        D = 1.0 + b * G
        y[r] = (h * S1[r] + y[r]) / D
        g[r] = G / D
        a[r] = b

    ends = [s[0] for s in steps[1:]] + [torch.empty(0, dtype=torch.int64, device=DEV)]
    nxt_Z = torch.zeros(n, dtype=torch.float64, device=DEV)
    for (r, q, Z), cont in zip(reversed(steps), reversed(ends)):
        sh = None if vel is None else sign * ((vel[q] - vel[org[r]]) @ d)
        cn, en = _optics(m, q, sh, ln, dx)
        if len(cont):  # rays that go on beyond this point: their next point's row comes first
            full = torch.empty(n, F, dtype=torch.float64, device=DEV)
            full[r] = cn
            Zr = torch.empty(n, dtype=torch.float64, device=DEV)
            Zr[r] = Z
            row(cont, full[cont], nxt_Z[cont] - Zr[cont])
        c1[r], S1[r] = cn, en / cn
        nxt_Z[r] = Z
    if steps:
        r = steps[0][0]
        row(r, co[r], nxt_Z[r])
    return a, g, y


def _solve(m, org, dirs, ln, dx):
    nbr = _padded(m)
    I = m["I_bc"][None, :]
    J = 0.0
    co, eo = _optics(m, org, None, ln, dx)
    w2 = 1.0 / len(dirs)
    for v in dirs:
        d = torch.tensor(v, dtype=torch.float64, device=DEV)
        sides, some = [], []
        for s in (1.0, -1.0):
            st = _walk(m, nbr, org, s * d)
            sides.append(_side(m, st, org, s * d, s, co, I, ln, dx))
            h = torch.zeros(len(org), dtype=torch.bool, device=DEV)
            if st:
                h[st[0][0]] = True
            some.append(h[:, None])
        (ap, gp, yp), (am, gm, ym) = sides
        h = 0.5 * (ap + am)
        both = (h * eo / co + yp + ym) / (h + gp + gm)
        # an empty side: its step is 0, its pivot 1 and its right-hand side the boundary's
        J = J + w2 * torch.where(some[0] | some[1], both, I.expand_as(both))
    return J


def exact(case, seed):
    c = case
    if c["kind"] in ("trace", "train", "adaptive") or c.get("dtau") or c.get("dv"):
        return None
    m = _inputs(case, seed)
    if c["kind"] == "infer":
        return _exact_infer(c, m)
    if c["kind"] != "batch" and work(case)["flops"] > 1.5e12:
        return None  # more than some 20 seconds in plain torch
    ln, dx, _ = _grid_x(c["blocks"], c["nf"])
    dirs = _directions(c["nside"])
    if c["kind"] == "batch":
        return [_solve(x, torch.arange(len(x["pos"]), device=DEV), dirs, ln, dx) for x in m]
    org = m["origins"].long() if c["kind"] == "compute" else torch.arange(len(m["pos"]), device=DEV)
    return _solve(m, org, dirs, ln, dx)


def _exact_infer(c, m):
    """Features, network and J = J1 exp(m) with nothing rounded but the inputs and the weights."""
    P, F = c["P"], c["nf"]
    w, W = m["w"].double(), []
    for shape in ((16, 256), (256,), (256, 256), (256,), (256, 256), (256,), (256, 2), (2,)):
        n = math.prod(shape)
        W.append(w[:n].reshape(shape))
        w = w[n:]
    nbr = _padded(m)
    mean, istd = (torch.tensor(m[k], dtype=torch.float64, device=DEV) for k in ("mean", "istd"))
    lc, S = m["chi"].double(), m["eta"].double() / m["chi"].double()
    Y = torch.empty(P * F, 2, dtype=torch.float64, device=DEV)
    for p0 in range(0, P, 2048):
        p = torch.arange(p0, min(P, p0 + 2048), device=DEV)
        k = nbr[p]
        ok = (k >= 0)[..., None]
        nd = ok.sum(1).double()
        kc = k.clamp_min(0)
        mean_n = lambda v: torch.where(ok, v, 0.0).sum(1) / nd  # noqa: E731
        cq, sq = lc[kc], S[kc]
        lq = cq.log()
        ml = mean_n(lq)
        rel = lambda f, fq: torch.where(ok, ((f[:, None] - fq) / (f[:, None] + fq)).abs(), 0.0).amax(1)  # noqa: E731
        L = mean_n((m["pos"][kc] - m["pos"][p][:, None]).norm(dim=-1, keepdim=True)).expand(-1, F)
        J1 = m["J1"][p].double()
        a = m["u"][p].double().clamp_min(1e-30).log() - J1.log()[:, None]
        f = torch.stack([J1.log(), lc[p].log(), S[p].log(), ml, mean_n(sq.log()),
                         mean_n((lq - ml[:, None]) ** 2).sqrt(), rel(lc[p], cq), rel(S[p], sq), L.log(),
                         (lc[p] * L).log(), (m["fx"].double() / 5.0).expand(len(p), F), nd.log().expand(-1, F),
                         a.amax(1), a.amin(1), (a - a.mean(1, keepdim=True)).square().mean(1).sqrt(),
                         torch.zeros_like(ml)], -1)
        h = ((f - mean) * istd).reshape(-1, 16)
        for i in (0, 2, 4):
            h = torch.nn.functional.silu(h @ W[i] + W[i + 1])
        Y[p0 * F:p0 * F + len(h)] = h @ W[6] + W[7]
    J = m["J1"].double() * Y[:, 0].reshape(P, F).exp()
    return dict(X=None, Y=Y, J=J)
