"""Performance cases: the work that a program using this package has it do.

Each case is one call path through the public Python entry points, from the
paper's smallest instance to the largest on-the-fly layout. A case is a dict
of plain values; `prepare` builds what such a program holds before the call
(inputs on the GPU, a solver handle), `run` makes one pass and returns its
outputs, `exact` computes the same outputs with plain FP64 torch.

Inputs are synthetic C-RAN layouts: devices uniform in a square with Gaussian
hot spots, RRHs on a jittered grid, lognormal traffic, rates of the downlink
model with lognormal shadowing, cost (1/R) / median(1/R).
"""

import ctypes
import math

import numpy as np
import torch

from paper_1805_01559_amd import ot_assoc as A

RADIO = dict(tx_power_w=1.0, ref_gain=10.0 ** -3.8, pathloss_exp=3.5, min_dist_m=10.0, shadow_sigma_db=8.0,
             noise_w=10.0 ** ((-174.0 + 10.0 * math.log10(20e6) - 30.0) / 10.0), bandwidth_hz=20e6)
CHUNK = 1 << 25  # cells of a cost evaluated at a time


def listed():
    return [
        # the smallest instance of the paper's run-time table (100 users, 25 RRHs), stopped at 0.1 %: one scheduling
        # instant of a small site, where launches and waits are everything
        dict(name="paper_100x25", kind="dense", I=100, J=25, side=500.0, eps=0.05, tol=1e-3, iters=10),
        # the quick-start of a program without torch: numpy arrays in, numpy plan out
        dict(name="host_1000x50", kind="host", I=1000, J=50, side=1000.0, eps=0.05, tol=1e-9, iters=35),
        # a planning study of Sec. IV: 25 RRHs, thousands of users, q from the maxSINR rule (Lemma 1), then the
        # queueing evaluation of the association
        dict(name="policy_rates_5000x25", kind="policy", I=5000, J=25, side=1000.0, eps=0.05, tol=1e-8, iters=40),
        # FP64 costs solved in FP64 throughout, to a tight tolerance (a reference run); ragged sizes
        dict(name="fp64_2999x197", kind="fp64", I=2999, J=197, side=2000.0, eps=0.02, tol=1e-10, iters=60),
        # the main workload: one scheduling instant of a large C-RAN, dense cost in HBM, plan in HBM
        dict(name="dense_20000x400", kind="dense", I=20000, J=400, side=5000.0, eps=0.02, tol=1e-8, iters=52),
        # the adaptive association (Alg. 2) over positions: up to eight warm-started solves
        dict(name="adaptive_geo_8000x150", kind="adaptive", I=8000, J=150, side=3000.0, eps=0.02, tol=1e-8, iters=250,
             outer=8),
        # the distance cost (choice (i) of Sec. IV): slow convergence, over a thousand iterations
        dict(name="euclid_20000x400", kind="euclid", I=20000, J=400, side=5000.0, eps=0.02, tol=1e-8, iters=1250),
        # a dense cost far above what the chip can hold: the streaming path
        dict(name="dense_200000x400", kind="dense", I=200000, J=400, side=5000.0, eps=0.02, tol=1e-8, iters=52),
        # the largest layout: the cost comes from the positions
        dict(name="geo_200000x2000", kind="geo", I=200000, J=2000, side=15000.0, eps=0.01, tol=1e-8, iters=67),
        # 256 uneven instances at once (many sites, one controller), with their plans
        dict(name="batch_256", kind="batch", n=256, sizes=3000, eps=0.05, tol=1e-6, iters=28),
        # a serving loop: layouts that drift a few metres per step, warm starts from the step before
        dict(name="serve_24x4", kind="serve", n=24, steps=4, sizes=4100, eps=0.02, tol=1e-6, iters=40),
        # 64 traffic snapshots of one layout on the matrix cores
        dict(name="snapshots_64", kind="snapshots", B=64, I=20000, J=400, side=5000.0, eps=0.02, tol=1e-6, iters=35),
    ]


def _log_int(rng, lo, hi):
    return int(min(hi, math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["dense", "dense", "dense", "host", "policy", "fp64", "adaptive", "euclid", "geo", "geo", "batch",
                       "serve", "snapshots"])
    if kind == "batch":
        return dict(kind=kind, n=_log_int(rng, 8, 256), sizes=rng.randrange(1, 1 << 20), eps=0.05, tol=1e-6, iters=28)
    if kind == "serve":
        return dict(kind=kind, n=_log_int(rng, 4, 32), steps=rng.randrange(2, 5), sizes=rng.randrange(1, 1 << 20),
                    eps=0.02, tol=1e-6, iters=40)
    eps, tol = rng.choice([0.02, 0.05]), rng.choice([1e-6, 1e-8])
    if kind == "dense":
        J = _log_int(rng, 20, 1500)
        I = _log_int(rng, 2 * J, min(200000, 80_000_000 // J))
    elif kind == "geo":
        J = _log_int(rng, 20, 1500)
        I = _log_int(rng, 2 * J, min(200000, 100_000_000 // J))
    elif kind == "policy":
        J = _log_int(rng, 4, 40)
        I = _log_int(rng, 60 * J, 20000)
    elif kind == "host":
        J = _log_int(rng, 20, 100)
        I = _log_int(rng, 2 * J, 5000)
    else:
        J = _log_int(rng, 20, 400)
        I = _log_int(rng, 2 * J, 20000)
    c = dict(kind=kind, I=I, J=J, side=float(int(250 * math.sqrt(J))), eps=eps, tol=tol, iters=50)
    if kind == "euclid":
        c.update(eps=0.05, iters=400)
    if kind == "fp64":
        c.update(tol=1e-10)
    if kind == "adaptive":
        c.update(outer=rng.randrange(3, 9), iters=200)
    if kind == "snapshots":
        c.update(B=_log_int(rng, 2, 64), eps=0.02, tol=1e-6)
    return c


# ------------------------------------------------------------------ inputs --

def _sizes(case):
    """(I, J) pairs of a batch or a serving loop, log-uniform."""
    r = np.random.Generator(np.random.PCG64(case["sizes"]))
    n = case["n"]
    I = np.exp(r.uniform(math.log(500), math.log(20001), n)).astype(int).clip(500, 20000)
    J = np.exp(r.uniform(math.log(20), math.log(401), n)).astype(int).clip(20, 400)
    return [(int(i), int(j)) for i, j in zip(I, J)]


class Layout:
    """Positions (float32, GPU), marginals (float64, GPU) and the shadowing key."""

    def __init__(self, I, J, side, seed):
        r = np.random.Generator(np.random.PCG64(seed))
        self.I, self.J, self.side = I, J, side
        self.key = int(r.integers(0, 2**62)) * 2 + 1
        rows = max(1, int(math.sqrt(J)))
        cols = -(-J // rows)
        k = np.arange(J)
        jit = r.uniform(-0.25, 0.25, (J, 2))
        rrh = np.stack([(k % cols + 0.5 + jit[:, 0]) * side / cols, (k // cols + 0.5 + jit[:, 1]) * side / rows], 1)
        hot = int(0.3 * I)
        dev = r.uniform(0.0, side, (I, 2))
        centres = r.uniform(0.1 * side, 0.9 * side, (4, 2))
        dev[:hot] = np.clip(centres[r.integers(0, 4, hot)] + r.normal(0.0, 0.04 * side, (hot, 2)), 0.0, side)
        lam = np.exp(r.standard_normal(I))
        self.xy = torch.from_numpy(dev.astype(np.float32)).cuda()
        self.rrh = torch.from_numpy(rrh.astype(np.float32)).cuda()
        self.a = torch.from_numpy(lam / lam.sum()).cuda()
        self.b = torch.full((J,), 1.0 / J, dtype=torch.float64, device="cuda")
        self.rng = r

    def move(self, metres):
        th = torch.from_numpy(self.rng.uniform(0.0, 2.0 * math.pi, self.I)).cuda()
        step = metres * torch.stack([th.cos(), th.sin()], 1)
        return (self.xy.double() + step).clamp(0.0, self.side).float()


def _shr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _i64(c):
    return c - (1 << 64) if c >= 1 << 63 else c


def _shadow(key, rows, J):
    """Standard normals of the links (rows x J): SplitMix64 of key ^ (i 2^32 + j), Box-Muller."""
    j = torch.arange(J, dtype=torch.int64, device=rows.device)
    x = ((rows[:, None] << 32) + j) ^ _i64(key)
    x = x + _i64(0x9E3779B97F4A7C15)
    x = (x ^ _shr(x, 30)) * _i64(0xBF58476D1CE4E5B9)
    x = (x ^ _shr(x, 27)) * _i64(0x94D049BB133111EB)
    x = x ^ _shr(x, 31)
    u1 = ((x >> 32) & 0xFFFFFFFF).double().add_(0.5).mul_(2.0**-32)
    u2 = (x & 0xFFFFFFFF).double().add_(0.5).mul_(2.0**-32)
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)


def _inv_rate_rows(xy, rrh, key, rows):
    """1 / R_ij in FP64 for the given device rows."""
    p = RADIO
    d = xy[rows].double()[:, None, :] - rrh.double()[None, :, :]
    d2 = (d * d).sum(2).clamp_(min=p["min_dist_m"] ** 2)
    pg = 10.0 ** (p["shadow_sigma_db"] * _shadow(key, rows, rrh.shape[0]) / 10.0) * d2 ** (-0.5 * p["pathloss_exp"])
    n0 = p["noise_w"] / (p["tx_power_w"] * p["ref_gain"])
    top, j1 = pg.max(1, keepdim=True)
    rest = pg.scatter(1, j1, 0.0).sum(1, keepdim=True)  # the interference of the strongest link, without cancellation
    den = (rest + top - pg + n0).scatter(1, j1, rest + n0)
    return math.log(2.0) / (p["bandwidth_hz"] * torch.log1p(pg / den))


def _rows(I, J):
    n = max(1, CHUNK // J)
    return [torch.arange(q, min(I, q + n), device="cuda") for q in range(0, I, n)]


def _scale(xy, rrh, key):
    """Lower median of 1/R over at most 2000 evenly spaced devices."""
    I = xy.shape[0]
    rows = torch.linspace(0, I - 1, min(I, 2000), device="cuda").long()
    return float(_inv_rate_rows(xy, rrh, key, rows).flatten().median())


def _inv_rate(L, xy=None):
    xy = L.xy if xy is None else xy
    return torch.cat([_inv_rate_rows(xy, L.rrh, L.key, r) for r in _rows(L.I, L.J)])


def _cost32(L):
    """Dense FP32 cost matrix of a layout."""
    s = _scale(L.xy, L.rrh, L.key)
    return torch.cat([(_inv_rate_rows(L.xy, L.rrh, L.key, r) / s).float() for r in _rows(L.I, L.J)])


def _layout(case, seed):
    return Layout(case["I"], case["J"], case["side"], seed)


# ----------------------------------------------------------------- prepare --

def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind == "batch":
        Ls = [Layout(I, J, 1000.0, seed * 1000 + k) for k, (I, J) in enumerate(_sizes(case))]
        s.update(costs=[_cost32(L) for L in Ls], a=[L.a for L in Ls], b=[L.b for L in Ls])
        s.update(solver=A.Solver(16, 16), plans=torch.empty(sum(L.I * L.J for L in Ls), device="cuda"))
        return s
    if kind == "serve":
        reqs, dims = [], []
        for k, (I, J) in enumerate(_sizes(case)):
            L = Layout(I, J, 1000.0, seed * 1000 + k)
            scale = _scale(L.xy, L.rrh, L.key)
            for t in range(case["steps"]):
                if t:
                    L.xy = L.move(5.0)
                reqs.append((t, k + 1, A.geometry_desc(L.xy, L.rrh, RADIO, L.key, scale), L.a, L.b))
            dims.append((I, J))
        reqs.sort(key=lambda q: (q[0], q[1]))
        s.update(reqs=reqs, dims=dims, server=A.Server())
        return s
    L = _layout(case, seed)
    I, J = L.I, L.J
    s.update(L=L, solver=A.Solver(I, J, precision=A.OT_PREC_FP64 if kind == "fp64" else A.OT_PREC_FP32))
    if kind == "host":
        s.update(C=_cost32(L).cpu().numpy(), a=L.a.cpu().numpy(), b=L.b.cpu().numpy())
    elif kind == "dense":
        s.update(C=_cost32(L), plan=torch.empty((I, J), device="cuda"))
    elif kind == "policy":
        s.update(R=(1.0 / _inv_rate(L)).float(), scale=_scale(L.xy, L.rrh, L.key),
                 plan=torch.empty((I, J), device="cuda"))
    elif kind == "fp64":
        s.update(C=_inv_rate(L) / _scale(L.xy, L.rrh, L.key),
                 plan=torch.empty((I, J), dtype=torch.float64, device="cuda"))
    elif kind in ("geo", "adaptive"):
        s.update(scale=_scale(L.xy, L.rrh, L.key), plan=torch.empty((I, J), device="cuda"))
    elif kind == "euclid":
        s.update(scale=_dist_scale(L), plan=torch.empty((I, J), device="cuda"))
    elif kind == "snapshots":
        s.update(C=_cost32(L), A=_snapshots(case, L))
        s.update(f=torch.empty((case["B"], I), dtype=torch.float64, device="cuda"),
                 g=torch.empty((case["B"], J), dtype=torch.float64, device="cuda"))
    return s


def _dist_rows(L, r):
    d = L.xy[r].double()[:, None, :] - L.rrh.double()[None, :, :]
    return (d * d).sum(2).sqrt()


def _dist_scale(L):
    rows = torch.linspace(0, L.I - 1, min(L.I, 2000), device="cuda").long()
    return float(_dist_rows(L, rows).flatten().median())


def _snapshots(case, L):
    lam = torch.from_numpy(np.exp(L.rng.standard_normal((case["B"], L.I)))).cuda()
    return (lam / lam.sum(1, keepdim=True)).contiguous()


# --------------------------------------------------------------------- run --

def _solved(res, plan):
    return dict(plan=plan, objective=res.objective, reg_objective=res.reg_objective, dual_objective=res.dual_objective)


def run(s):
    kind, c = s["kind"], s["case"]
    if kind == "batch":
        _, res = s["solver"].solve_batch(s["costs"], s["a"], s["b"], c["eps"], c["tol"])
        o = 0
        for k, C in enumerate(s["costs"]):
            p = ctypes.c_void_p(s["plans"].data_ptr() + 4 * o)
            A.ot_assoc_batch_plan(s["solver"].h, k, p, A.OT_MEM_DEVICE, A.OT_F32)
            o += C.numel()
        return dict(plans=s["plans"], objective=torch.tensor([r.objective for r in res]))
    if kind == "serve":
        return _run_serve(s, c)
    S, L = s["solver"], s["L"]
    if kind == "host":
        _, res = S.solve_dense(s["C"], s["a"], s["b"], c["eps"], c["tol"])
        return _solved(res, S.plan(dtype=np.float32))
    if kind == "policy":
        d = A.matrix_desc(s["R"], A.OT_COST_RATES, s["scale"])
        assoc, lam = S.maxsinr(*d, L.a)
        b = torch.from_numpy(lam).cuda()
        _, res = S.solve_rates(s["R"], s["scale"], L.a, b, c["eps"], c["tol"])
        S.plan(s["plan"])
        rho, en, ev = S.evaluate(0.25 * L.J, 1.0)
        return dict(_solved(res, s["plan"]), assoc=assoc, Lambda=lam, rho=rho.astype(np.float32),
                    jobs=en.astype(np.float32), mean_completion=ev.mean_completion)
    if kind == "snapshots":
        _, res = S.solve_snapshots(s["C"], s["A"], L.b, c["eps"], c["tol"])
        f, g = s["f"], s["g"]
        for q in range(c["B"]):
            A.ot_assoc_snapshot_potentials(S.h, q, ctypes.c_void_p(f[q].data_ptr()), ctypes.c_void_p(g[q].data_ptr()),
                                           A.OT_MEM_DEVICE)
        # prices relative to the first RRH (potentials are defined up to a constant), handed on in 32 bits
        return dict(f=(f + g[:, :1]).float(), g=(g - g[:, :1]).float(),
                    objective=torch.tensor([r.objective for r in res]))
    if kind == "adaptive":
        d = A.geometry_desc(L.xy, L.rrh, RADIO, L.key, s["scale"])
        _, q, js, r = S.adaptive(*d, L.a, c["eps"], c["tol"], max_outer=c["outer"])
        return dict(plan=S.plan(s["plan"]), q=q, jstar=np.pad(js, (0, c["outer"] - len(js)), constant_values=-1),
                    max_load=r.max_load)
    if kind == "geo":
        S.set_plan_output(s["plan"])
        _, res = S.solve_geometry(L.xy, L.rrh, RADIO, L.key, s["scale"], L.a, L.b, c["eps"], c["tol"])
    elif kind == "euclid":
        S.set_plan_output(s["plan"])
        _, res = S.solve_euclid(L.xy, L.rrh, s["scale"], L.a, L.b, c["eps"], c["tol"], max_iter=5000)
    else:
        S.set_plan_output(s["plan"])
        _, res = S.solve_dense(s["C"], L.a, L.b, c["eps"], c["tol"])
    return _solved(res, S.plan(s["plan"]))


def _run_serve(s, c):
    srv, objective = s["server"], {}
    todo, nxt = s["reqs"], 0
    for t in range(c["steps"]):
        sent = 0
        while nxt < len(todo) and todo[nxt][0] == t:
            _, key, d, a, b = todo[nxt]
            srv.submit(d, a, b, c["eps"], c["tol"], 2000, layout_key=key, user_tag=nxt)
            nxt += 1
            sent += 1
        while sent:
            for done in srv.progress():
                objective[done.user_tag] = done.result.objective
                sent -= 1
    f, g = [], []
    for k, (I, J) in enumerate(s["dims"]):
        fk, gk = srv.potentials(k + 1, I, J)
        f.append((fk + gk[0]).astype(np.float32))
        g.append((gk - gk[0]).astype(np.float32))
    return dict(f=np.concatenate(f), g=np.concatenate(g),
                objective=torch.tensor([objective[q] for q in range(len(todo))]))


# -------------------------------------------------------------------- work --

def work(case):
    """Bytes: every input read once, every output written once. Flops: two multiply-adds per cell and iteration (the
    row and the column sum of the scaling form), for the iterations such an instance takes."""
    kind, it = case["kind"], case["iters"]
    if kind in ("batch", "serve"):
        cells = sum(I * J for I, J in _sizes(case))
        steps = case.get("steps", 1)
        vec = sum(8 * (I + J) for I, J in _sizes(case))
        return dict(bytes=(8 * cells if kind == "batch" else 0) + 2 * steps * vec, flops=4.0 * cells * it * steps)
    I, J = case["I"], case["J"]
    cells, vec = I * J, 8 * (I + J)
    if kind == "snapshots":
        return dict(bytes=4 * cells + 2 * case["B"] * vec, flops=4.0 * cells * it * case["B"])
    size = 16 if kind == "fp64" else 4 if kind in ("geo", "euclid", "adaptive") else 8  # cost in (if any), plan out
    return dict(bytes=size * cells + 2 * vec, flops=4.0 * cells * it)


# ------------------------------------------------------------------- exact --

def _solve64(C, a, b, eps, g=None, most=8000):
    """Potentials of the converged Sinkhorn iteration in FP64 (from g, else g = 0)."""
    g = torch.zeros_like(b) if g is None else g
    la, lb = a.log(), b.log()
    for _ in range(2):  # log domain: no column can underflow
        f = eps * (la - torch.logsumexp((g - C) / eps, 1))
        g = eps * (lb - torch.logsumexp((f[:, None] - C) / eps, 0))
    done, n, last = 0, 1, math.inf
    while done < most:
        K = torch.exp((f[:, None] + g - C) / eps)
        Kt = K.t().contiguous()
        u, v = torch.ones_like(a), torch.ones_like(b)
        for _ in range(n):
            u = a / (K @ v)
            v = b / (Kt @ u)
        f, g = f + eps * u.log(), g + eps * v.log()
        r = float((u * (K @ v) - a).abs().sum())
        done += n
        if r < 1e-12 or (r < 1e-10 and r > 0.9 * last):  # converged, or as far as the rounding of the sums lets it
            break
        n, last = min(40, 2 * n), r
    return f, g


def _stats64(C, f, g, a, b, eps):
    pi = torch.exp((f[:, None] + g - C) / eps)
    obj = float((C * pi).sum())
    ent = float((pi * ((f[:, None] + g - C) / eps - 1.0)).sum())
    return pi, dict(objective=obj, reg_objective=obj + eps * ent,
                    dual_objective=float(f @ a + g @ b - eps * pi.sum()))


def exact(case, seed):
    kind, eps = case["kind"], case["eps"]
    if kind == "batch":
        plans, obj = [], []
        for k, (I, J) in enumerate(_sizes(case)):
            L = Layout(I, J, 1000.0, seed * 1000 + k)
            C = _cost32(L).double()
            pi, st = _stats64(C, *_solve64(C, L.a, L.b, eps), L.a, L.b, eps)
            plans.append(pi.flatten().float() if case["n"] > 400 else pi.flatten())
            obj.append(st["objective"])
        return dict(plans=torch.cat(plans), objective=torch.tensor(obj, dtype=torch.float64))
    if kind == "serve":
        fs, gs, obj = [], [], {}
        n = case["n"]
        for k, (I, J) in enumerate(_sizes(case)):
            L = Layout(I, J, 1000.0, seed * 1000 + k)
            scale = _scale(L.xy, L.rrh, L.key)
            g = None
            for t in range(case["steps"]):
                if t:
                    L.xy = L.move(5.0)
                C = (_inv_rate(L) / scale).float().double()
                f, g = _solve64(C, L.a, L.b, eps, g)
                obj[t * n + k] = _stats64(C, f, g, L.a, L.b, eps)[1]["objective"]
            fs.append(f + g[0])
            gs.append(g - g[0])
        return dict(f=torch.cat(fs), g=torch.cat(gs),
                    objective=torch.tensor([obj[q] for q in range(n * case["steps"])], dtype=torch.float64))
    L = _layout(case, seed)
    if kind in ("dense", "host", "snapshots"):
        C = _cost32(L).double()
    elif kind == "euclid":
        C = torch.cat([_dist_rows(L, r) for r in _rows(L.I, L.J)]) / _dist_scale(L)
    elif kind == "policy":
        C = 1.0 / (1.0 / _inv_rate(L)).float().double() / _scale(L.xy, L.rrh, L.key)
    else:
        C = _inv_rate(L) / _scale(L.xy, L.rrh, L.key)
    if kind == "snapshots":
        fs, gs, obj = [], [], []
        for a in _snapshots(case, L):
            f, g = _solve64(C, a, L.b, eps)
            fs.append(f + g[0])
            gs.append(g - g[0])
            obj.append(float((C * torch.exp((f[:, None] + g - C) / eps)).sum()))
        return dict(f=torch.stack(fs), g=torch.stack(gs), objective=torch.tensor(obj, dtype=torch.float64))
    if kind == "policy":
        near = C.min(1).indices
        b = torch.zeros_like(L.b).index_add_(0, near, L.a)
        f, g = _solve64(C, L.a, b, eps)
        pi, st = _stats64(C, f, g, L.a, b, eps)
        rho = 0.25 * L.J * (C * pi).sum(0)
        T = (C * pi / (1.0 - rho)).sum(1) / L.a
        return dict(st, plan=pi, assoc=near, Lambda=b, rho=rho, jobs=rho / (1.0 - rho),
                    mean_completion=float(T.mean()))
    if kind == "adaptive":
        return _adaptive64(case, C, L.a, eps)
    f, g = _solve64(C, L.a, L.b, eps)
    pi, st = _stats64(C, f, g, L.a, L.b, eps)
    return dict(st, plan=pi)


def _adaptive64(case, C, a, eps):
    J = C.shape[1]
    q = torch.full((J,), float(a.sum()) / J, dtype=torch.float64, device=C.device)
    delta = 0.01 * float(a.sum()) / J
    best, js, g = None, [], None
    for _ in range(case["outer"]):
        f, g = _solve64(C, a, q, eps, g)
        pi = torch.exp((f[:, None] + g - C) / eps)
        load = (C * pi).sum(0)
        j = int(load.argmax())
        js.append(j)
        if best is None or float(load[j]) < best[0]:
            best = (float(load[j]), q.clone(), pi)
        else:
            break
        if float(q[j]) - delta <= 0.0:
            break
        q = q + delta / (J - 1)
        q[j] -= delta + delta / (J - 1)
    js += [-1] * (case["outer"] - len(js))
    return dict(plan=best[2], q=best[1], jstar=torch.tensor(js), max_load=best[0])
