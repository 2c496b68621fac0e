"""Performance cases of the batched safety filter: the calls a program makes through SafetyFilter,
project_differentiable, qp_equality_differentiable and Batch, over the sizes of the repository's
workloads and of its tests.

Each case is a dict of plain values; `prepare` makes its inputs on the GPU from a seed, `run` is one
pass, `work` what a pass cannot do without, and `exact` the same outputs in 64 bits from plain torch.

Kinds of case:
  solve   one problem, a batch of sampled trajectories through the filter (sf_project)
  ragged  many problems of mixed swarm sizes in one persistent, graph-replayed call
  train   forward with checkpoints, the loss of a warm-start network, and its gradients
  layer   the decoders' equality-only QP layer, forward and reverse
  check   FP64 constraint violations of a batch of trajectories
"""
import functools
import math

import numpy as np
import torch

from paper_2501_19042_amd import Batch, SafetyFilter
from paper_2501_19042_amd.sf import project_differentiable, qp_equality_differentiable
from workloads import SwarmConfig

SEP = 0.3                       # centre-to-centre safety distance (m)
BOX = (3.0, 3.0, 1.0)           # half sizes of the box of starts and goals (m)
RAGGED_SIZES = (8, 16, 32)


def listed():
    return [
        # A planner that asks for one small swarm's next plan: four candidates, few iterations, and
        # the per-sample status that it selects by.  Latency of the whole call.
        {"name": "plan_8_robots", "kind": "solve", "robots": 8, "dims": 3, "degree": 10, "horizon": 100,
         "samples": 4, "iters": 100, "precision": "fp32", "workspace": False, "warm": False, "resid": False,
         "status": True},
        # The 4-robot crossing in the plane, 8 samples, 200 iterations in FP64.
        {"name": "circle_4_robots_2d", "kind": "solve", "robots": 4, "dims": 2, "degree": 10, "horizon": 100,
         "samples": 8, "iters": 200, "precision": "fp64", "workspace": False, "warm": False, "resid": True,
         "status": False},
        # The 16-robot batch of 1024 samples at 300 iterations in the 16-bit form: trajectories and
        # multipliers, without the residual report.
        {"name": "swarm_16", "kind": "solve", "robots": 16, "dims": 3, "degree": 10, "horizon": 100,
         "samples": 1024, "iters": 300, "precision": "bf16", "workspace": False, "warm": False, "resid": False,
         "status": False},
        # A re-plan from the last solution and its multipliers inside a workspace: odd sizes of
        # swarm, polynomial and horizon, a batch that does not fill the chip.
        {"name": "replan_13", "kind": "solve", "robots": 13, "dims": 3, "degree": 9, "horizon": 75,
         "samples": 333, "iters": 60, "precision": "fp16", "workspace": True, "warm": True, "resid": True,
         "status": False},
        # Reference solutions of the 16-robot problem in FP64.
        {"name": "reference_16_fp64", "kind": "solve", "robots": 16, "dims": 3, "degree": 10, "horizon": 100,
         "samples": 64, "iters": 150, "precision": "fp64", "workspace": False, "warm": False, "resid": True,
         "status": False},
        # The 32-robot batch: degree 12, 120 steps, 4096 samples, 300 iterations.
        {"name": "swarm_32", "kind": "solve", "robots": 32, "dims": 3, "degree": 12, "horizon": 120,
         "samples": 4096, "iters": 300, "precision": "bf16", "workspace": False, "warm": False, "resid": False,
         "status": False},
        # A server's queue: problems of 8, 16 and 32 robots with 1..256 samples each, one call.
        {"name": "ragged_150_problems", "kind": "ragged", "problems": 150, "most": 256, "iters": 150,
         "precision": "fp32", "resid": True},
        # Training an initialisation of the 16-robot filter: 512 samples, 100 unrolled iterations.
        {"name": "train_16", "kind": "train", "robots": 16, "degree": 10, "horizon": 100, "samples": 512,
         "iters": 100, "every": 10, "workspace": False},
        # The same with more robots, inside a workspace, on a small batch.
        {"name": "train_24_workspace", "kind": "train", "robots": 24, "degree": 11, "horizon": 80, "samples": 48,
         "iters": 40, "every": 8, "workspace": True},
        # A decoder's training step over a small batch: the layer forward and reverse.
        {"name": "layer_batch", "kind": "layer", "robots": 16, "degree": 10, "samples": 64, "precision": "fp32"},
        # The layer over a whole data set of decoded trajectories.
        {"name": "layer_large", "kind": "layer", "robots": 16, "degree": 10, "samples": 1 << 19,
         "precision": "fp32"},
        # Feasibility of a batch of filtered trajectories.
        {"name": "check_16", "kind": "check", "robots": 16, "degree": 10, "horizon": 100, "samples": 1024,
         "precision": "fp32"},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "solve", "ragged", "train", "train", "layer", "check"])
    if kind == "ragged":
        form, iters = rng.choice(["fp32", "bf16", "fp16"]), rng.randint(50, 300)
        return {"kind": kind, "problems": _log(rng, 10, 150), "most": _log(rng, 8, 256), "iters": iters,
                "precision": form, "resid": form == "fp32" and iters <= 150}
    if kind == "train":
        ws = rng.random() < 0.3
        n = rng.randint(4, 16) if not ws and rng.random() < 0.7 else rng.randint(4, 28)
        large = n > 16 or ws
        return {"kind": kind, "robots": n, "degree": rng.randint(8, 13), "horizon": rng.randint(40, 100 if large else 120),
                "samples": _log(rng, 4, 64 if large else 512), "iters": rng.randint(15, 32 if large else 60),
                "every": rng.randint(4, 12), "workspace": ws}
    if kind == "layer":
        return {"kind": kind, "robots": rng.randint(2, 32), "degree": rng.randint(7, 14),
                "samples": _log(rng, 1, 1 << 17), "precision": rng.choice(["fp32", "fp32", "fp64"])}
    if kind == "check":
        return {"kind": kind, "robots": rng.randint(2, 32), "degree": rng.randint(7, 13),
                "horizon": rng.randint(30, 160), "samples": _log(rng, 1, 2048),
                "precision": rng.choice(["fp32", "fp64"])}
    form = rng.choice(["fp32", "fp32", "bf16", "bf16", "fp16", "fp64"])
    planar = form == "fp64" and rng.random() < 0.5
    n = rng.randint(3, 6) if planar else rng.randint(4, 16) if form == "fp64" else rng.randint(4, 32)
    # FP64 batches are reference runs: few samples and iterations
    horizon, iters = rng.randint(30, 160), rng.randint(25, 100 if form == "fp64" else 300)
    samples = _log(rng, 1, 64 if form == "fp64" else 2048 if n > 16 else 4096)
    return {"kind": kind, "robots": n, "dims": 2 if planar else 3, "degree": rng.randint(7, 13), "horizon": horizon,
            "samples": samples, "iters": iters, "precision": form,
            "workspace": not planar and rng.random() < 0.25, "warm": rng.random() < 0.3,
            # a residual report of few iterations or of a reference run; the status of a few candidates
            "resid": form == "fp64" or (form != "bf16" and iters <= 60),
            "status": samples <= 16 and rng.random() < 0.5}


# --- inputs ----------------------------------------------------------------------------------

def _config(robots, dims, degree, horizon, workspace):
    # the semi-axes of the workspace just hold the box of starts and goals
    ws = {"ws_a": 4.8, "ws_b": 2.2} if workspace else {}
    return SwarmConfig(n_robots=robots, dims=dims, degree=degree, horizon=horizon, t_final=10.0 if dims == 3 else 5.0,
                       safety_a=SEP, safety_b=SEP, vmax=1.5, amax=2.0, **ws)


def _configs(case):
    if case["kind"] == "ragged":
        return [_config(n, 3, 10, 100, False) for n in RAGGED_SIZES]
    return [_config(case["robots"], case.get("dims", 3), case["degree"], case.get("horizon", 100),
                    case.get("workspace", False))]


def _entries(case, seed):
    """(config, samples) of each problem."""
    if case["kind"] != "ragged":
        return [(0, case["samples"])]
    # the same numbers of samples for every seed, in another order
    u = np.random.default_rng([case["problems"], case["most"]]).random(case["problems"])
    counts = np.maximum(1, np.minimum(case["most"], np.floor(np.exp(u * math.log(case["most"] + 1)))).astype(int))
    order = np.random.default_rng([seed, 1]).permutation(case["problems"])
    return [(int(k % len(RAGGED_SIZES)), int(counts[k])) for k in order]


def _ends(cfg, r):
    """Starts and goals of one problem: a box with a minimum separation, goals a permutation of the
    starts (3D); a circle with antipodal goals (2D)."""
    n = cfg.n_robots
    if cfg.dims == 2:
        th = 2 * np.pi * np.arange(n) / n
        p = 2.0 * np.stack([np.cos(th), np.sin(th)], 1)
        return p, -p
    pts = np.zeros((0, 3))
    half = np.array(BOX)
    while len(pts) < n:
        p = half * (2 * r.random(3) - 1)
        if not len(pts) or ((pts - p) ** 2).sum(1).min() >= 0.25:
            pts = np.concatenate([pts, p[None]])
    return pts, pts[r.permutation(n)]


def _inputs(case, seed):
    """Sampled coefficients (straight lines between the ends plus noise on every coefficient) and
    boundary values at rest, both packed over the problems: float64 on the GPU."""
    cfgs = _configs(case)
    r = np.random.default_rng([seed, 2])
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 2 + 1)
    xs, bs = [], []
    for slot, count in _entries(case, seed):
        cfg = cfgs[slot]
        s, e = _ends(cfg, r)
        k = np.arange(cfg.degree + 1) / cfg.degree
        line = torch.from_numpy(s[:, :, None] + k * (e - s)[:, :, None]).cuda()
        sigma = 0.3 if cfg.dims == 2 else 0.4
        noise = torch.randn((count,) + tuple(line.shape), generator=g, device="cuda", dtype=torch.float32)
        xs.append(torch.add(line.float(), noise, alpha=sigma).reshape(-1))
        b = np.zeros(s.shape + (6,))
        b[:, :, 0], b[:, :, 3] = s, e
        bs.append(torch.from_numpy(b).reshape(-1))
    x = xs[0] if len(xs) == 1 else torch.cat(xs)
    b = torch.cat(bs).float().cuda()     # values that are the same in every precision
    return cfgs, x, b, g


def _dtype(case):
    return torch.float64 if case.get("precision") == "fp64" else torch.float32


def _make(case, seed):
    cfgs, x, b, g = _inputs(case, seed)
    dt = _dtype(case)
    st = {"case": case, "cfgs": cfgs}
    if case["kind"] == "ragged":
        st["x"], st["b"], st["entries"] = x.to(dt), b.to(dt), _entries(case, seed)
        return st
    c = cfgs[0]
    shape = (case["samples"], c.n_robots, c.dims, c.degree + 1)
    st["x"], st["b"] = x.reshape(shape).to(dt), b.reshape(c.n_robots, c.dims, 6).to(dt)

    def noise(scale):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(scale).to(dt)

    if case["kind"] == "layer":
        st["g"] = noise(1.0)
    elif case.get("warm") or case["kind"] == "train":
        # what a network or the last plan proposes: near the samples, with small multipliers
        st["xi0"], st["lam0"] = st["x"] + noise(0.1), noise(0.05)
    return st


def prepare(case, seed):
    st = _make(case, seed)
    st["sf"] = SafetyFilter(st["cfgs"])
    if case["kind"] == "ragged":
        st["batch"] = Batch(st["entries"])
        n = st["batch"].n_samples
        st["out"] = (torch.empty_like(st["x"]), torch.empty_like(st["x"]),
                     torch.empty((n, 2), dtype=st["x"].dtype, device="cuda") if case["resid"] else None, None, None)
    if case["kind"] == "train":
        for k in ("xi0", "lam0", "x"):
            st[k].requires_grad_(True)
    if case["kind"] == "layer":
        st["x"].requires_grad_(True)
        st["b"].requires_grad_(True)
    return st


def run(st):
    case, sf = st["case"], st["sf"]
    if case["kind"] == "solve":
        r = sf.project(st["x"], st["b"], case["iters"], precision=case["precision"], xi0=st.get("xi0"),
                       lam0=st.get("lam0"), want_resid=case["resid"], want_status=case["status"])
        return [r.xi, r.lam] + ([r.resid] if case["resid"] else []) + ([r.status] if case["status"] else [])
    if case["kind"] == "ragged":
        r = sf.project(st["x"], st["b"], case["iters"], batch=st["batch"], precision=case["precision"], graph=True,
                       persistent=True, out=st["out"])
        return [r.xi, r.lam] + ([r.resid] if case["resid"] else [])
    if case["kind"] == "train":
        xi, lam, res, fpr = project_differentiable(sf, st["x"], st["b"], case["iters"], st["xi0"], st["lam0"],
                                                   ckpt_every=case["every"])
        loss = (fpr + res).sum() + (xi - st["x"]).square().sum()
        return [xi.detach(), fpr.detach()] + list(torch.autograd.grad(loss, (st["xi0"], st["lam0"], st["x"])))
    if case["kind"] == "layer":
        y = qp_equality_differentiable(sf, st["x"], st["b"], precision=case["precision"])
        return [y.detach()] + list(torch.autograd.grad(y, (st["x"], st["b"]), st["g"]))
    return [sf.feasibility(st["x"], st["b"], precision=case["precision"])]


# --- what a pass cannot do without ---------------------------------------------------------------

def _iteration_flops(c):
    """One iteration of one sample: basis evaluation, back-projection to the free coefficients, the
    structured QP step, pair projections and bound balls."""
    n, D, m, H, mf = c.n_robots, c.dims, c.degree + 1, c.horizon, c.degree - 5
    pairs = n * (n - 1) // 2
    return (6 * n * D * H * (m + mf) + 4 * n * D * mf * mf + pairs * H * (19 + 2 * D) + 32 * n * H
            + (12 * n * H if c.ws_a > 0 else 0))


def work(case):
    cfgs = _configs(case)
    word = 8 if _dtype(case) == torch.float64 else 4
    nbytes = flops = 0
    for slot, count in _entries(case, 0):
        c = cfgs[slot]
        coef = c.n_robots * c.dims * (c.degree + 1)
        if case["kind"] == "layer":
            nbytes += count * coef * 4 * word
            flops += count * c.n_robots * c.dims * 6
        elif case["kind"] == "check":
            nbytes += count * (coef * word + 40)
            flops += count * _iteration_flops(c) // 2
        elif case["kind"] == "train":
            nbytes += count * coef * 8 * word
            flops += 4 * count * case["iters"] * _iteration_flops(c)
        else:
            nbytes += count * (coef * (5 if case.get("warm") else 3) + 2) * word
            flops += count * case["iters"] * _iteration_flops(c)
    return {"bytes": nbytes, "flops": flops}


# --- the same in 64 bits, from the method's equations ------------------------------------------

def _bern(N, k, t):
    return math.comb(N, k) * t ** k * (1 - t) ** (N - k) if 0 <= k <= N else np.zeros_like(t)


def _bases(c):
    N, t = c.degree, np.arange(c.horizon) / (c.horizon - 1)
    P = np.stack([_bern(N, k, t) for k in range(N + 1)], 1)
    V = np.stack([N / c.t_final * (_bern(N - 1, k - 1, t) - _bern(N - 1, k, t)) for k in range(N + 1)], 1)
    A = np.stack([N * (N - 1) / c.t_final ** 2 * (_bern(N - 2, k - 2, t) - 2 * _bern(N - 2, k - 1, t)
                                                   + _bern(N - 2, k, t)) for k in range(N + 1)], 1)
    return P, V, A


@functools.lru_cache(maxsize=8)
def _system(c):
    """Bases, pair incidence, and the blocks of the inverse of the KKT matrix of one axis."""
    P, V, A = _bases(c)
    n, m = c.n_robots, c.degree + 1
    ii, jj = np.triu_indices(n, 1)
    inc = np.zeros((len(ii), n))
    inc[np.arange(len(ii)), ii] = 1
    inc[np.arange(len(ii)), jj] = -1
    eye = np.eye(n)
    own = P.T @ P * (1.0 if c.ws_a > 0 else 0.0) + V.T @ V + A.T @ A
    Q = np.eye(n * m) + np.kron(inc.T @ inc, P.T @ P) + np.kron(eye, own)
    ends = np.kron(eye, np.stack([P[0], V[0], A[0], P[-1], V[-1], A[-1]]))
    K = np.block([[Q, ends.T], [ends, np.zeros((6 * n, 6 * n))]])
    inv = np.linalg.inv(K)[:n * m]
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    return {"P": t(P), "V": t(V), "A": t(A), "inc": t(inc), "ii": t(ii), "jj": t(jj), "free": t(inv[:, :n * m]),
            "bnd": t(inv[:, n * m:])}


def _residuals(c, s, xi):
    """F xi - e of each block: pair rows, velocity, acceleration and workspace rows, [S, rows, D, H]."""
    X, V, A = (torch.matmul(xi, s[k].T) for k in ("P", "V", "A"))
    scale = torch.tensor([1 / c.safety_a, 1 / c.safety_a, 1 / c.safety_b][:c.dims], device="cuda", dtype=xi.dtype)
    r = X[:, s["ii"]] - X[:, s["jj"]]
    d = torch.linalg.vector_norm(r * scale[:, None], dim=2, keepdim=True)
    rc = r * (1 - 1 / d).clamp(max=0)

    def ball(v, lim):
        return v * (1 - lim / torch.linalg.vector_norm(v, dim=2, keepdim=True).clamp(min=1e-300)).clamp(min=0)

    rw = None
    if c.ws_a > 0:
        w = torch.tensor([1 / c.ws_a, 1 / c.ws_a, 1 / c.ws_b][:c.dims], device="cuda", dtype=xi.dtype)
        q = torch.linalg.vector_norm(X * w[:, None], dim=2, keepdim=True)
        rw = X * (1 - 1 / q.clamp(min=1e-300)).clamp(min=0)
    return (r, V, A, X), (rc, ball(V, c.vmax), ball(A, c.amax), rw)


def _step(c, s, xb, b, xi, lam):
    """One fixed-point iteration: (xi, lambda) and the targets of the residual blocks; b [1 or S, n, D, 6]."""
    Y, R = _residuals(c, s, xi)
    S, n, D, m = xi.shape

    def back(r):
        pair = torch.matmul(s["inc"].T, r[0].reshape(S, -1, D * c.horizon)).reshape(S, n, D, c.horizon)
        g = torch.matmul(pair, s["P"]) + torch.matmul(r[1], s["V"]) + torch.matmul(r[2], s["A"])
        return g if r[3] is None else g + torch.matmul(r[3], s["P"])

    lam = lam - back(R)
    E = tuple(None if r is None else y - r for y, r in zip(Y, R))
    eta = (back(E) + lam + xb).permute(0, 2, 1, 3).reshape(S, D, n * m)
    z = torch.matmul(eta, s["free"].T) + torch.matmul(b.permute(0, 2, 1, 3).reshape(-1, D, n * 6), s["bnd"].T)
    return z.reshape(S, D, n, m).permute(0, 2, 1, 3), lam, E


def _primal(c, s, xi, E):
    X, V, A = (torch.matmul(xi, s[k].T) for k in ("P", "V", "A"))
    Y = (X[:, s["ii"]] - X[:, s["jj"]], V, A, X)
    sq = [(y - e).square().sum(2).flatten(1) for y, e in zip(Y, E) if e is not None]
    return sum(q.sum(1) for q in sq), torch.stack([q.amax(1) for q in sq]).amax(0).sqrt()


def _solve64(c, x, b, iters, xi0, lam0):
    s = _system(c)
    per = max(1, int(6e7 / (c.n_robots ** 2 * c.horizon)))
    out = []
    for k in range(0, x.shape[0], per):
        xb = x[k:k + per]
        xi = xb if xi0 is None else xi0[k:k + per]
        lam = torch.zeros_like(xb) if lam0 is None else lam0[k:k + per]
        bk = b[k:k + per] if b.shape[0] > 1 else b
        E = None
        for _ in range(iters):
            xi, lam, E = _step(c, s, xb, bk, xi, lam)
        ss, mx = _primal(c, s, xi, E)
        out.append((xi, lam, torch.stack([ss, mx], 1)))
    return [torch.cat(v).contiguous() for v in zip(*out)]


def _train64(c, case, st):
    s = _system(c)
    per = max(1, int(4e7 / (c.n_robots ** 2 * c.horizon)))
    out = []
    for k in range(0, case["samples"], per):
        xb, xi0, lam0 = (st[q][k:k + per].double().requires_grad_(True) for q in ("x", "xi0", "lam0"))
        keep, xi, lam, fpr = [], xi0.detach(), lam0.detach(), 0.0
        b = st["b"].double()[None]
        with torch.no_grad():
            for _ in range(case["iters"]):
                keep.append((xi, lam))
                xn, ln, E = _step(c, s, xb, b, xi, lam)
                fpr = fpr + ((xn - xi) ** 2).sum((1, 2, 3)) + ((ln - lam) ** 2).sum((1, 2, 3))
                xi, lam = xn, ln
        gx, gl = 2 * (xi - xb.detach()), torch.zeros_like(lam)
        gb = -gx
        for k2 in reversed(range(case["iters"])):
            with torch.enable_grad():
                p, q, xv = (v.detach().requires_grad_(True) for v in (*keep[k2], xb))
                xn, ln, E = _step(c, s, xv, b, p, q)
                obj = ((xn - p) ** 2).sum() + ((ln - q) ** 2).sum() + (xn * gx).sum() + (ln * gl).sum()
                if k2 == case["iters"] - 1:
                    obj = obj + _primal(c, s, xn, E)[0].sum()
                gx, gl, g3 = torch.autograd.grad(obj, (p, q, xv))
            gb = gb + g3
        out.append((xi, fpr, gx, gl, gb))
    return [torch.cat(v).contiguous() for v in zip(*out)]


def exact(case, seed):
    st = _make(case, seed)
    cfgs, x, b = st["cfgs"], st["x"], st["b"].double()
    c = cfgs[0]
    if case["kind"] == "layer":
        P, V, A = _bases(c)
        at = [0, 1, 2, c.degree - 2, c.degree - 1, c.degree]
        inv = torch.from_numpy(np.linalg.inv(np.stack([P[0], V[0], A[0], P[-1], V[-1], A[-1]])[:, at])).cuda()
        y, g = x.double(), st["g"].double()
        y[..., at] = torch.matmul(b, inv.T)
        gb = torch.matmul(g[..., at].sum(0), inv)
        g[..., at] = 0
        return [y, g, gb]
    if case["kind"] == "check":
        s = _system(c)
        out = []
        for k in range(0, case["samples"], 128):
            xi = x[k:k + 128].double()
            X, V, A = (torch.matmul(xi, s[q].T) for q in ("P", "V", "A"))
            r = torch.linalg.vector_norm(X[:, s["ii"]] - X[:, s["jj"]], dim=2).flatten(1).amin(1)
            rows = torch.stack([s["P"][0], s["V"][0], s["A"][0], s["P"][-1], s["V"][-1], s["A"][-1]])
            out.append(torch.stack([c.safety_a - r, torch.linalg.vector_norm(V, dim=2).flatten(1).amax(1) - c.vmax,
                                    torch.linalg.vector_norm(A, dim=2).flatten(1).amax(1) - c.amax,
                                    (torch.matmul(xi, rows.T) - b).abs().flatten(1).amax(1), torch.zeros_like(r)], 1))
        return [torch.cat(out)]
    if case["kind"] == "train":
        return _train64(c, case, st)
    if case["kind"] == "solve":
        d = lambda k: st[k].double() if k in st else None  # noqa: E731
        if case["robots"] ** 2 * case["horizon"] * case["samples"] * case["iters"] > 3e12:
            return None     # over about 20 seconds
        xi, lam, res = _solve64(c, x.double(), b[None], case["iters"], d("xi0"), d("lam0"))
        return [xi, lam] + ([res] if case["resid"] else []) + ([None] if case["status"] else [])
    # ragged: all samples of one swarm size together, then back into the order of the problems
    parts, o, ob = [], 0, 0
    for slot, count in st["entries"]:
        n, m = cfgs[slot].n_robots, cfgs[slot].degree + 1
        parts.append((slot, x[o:o + count * n * 3 * m].reshape(count, n, 3, m).double(),
                      b[ob:ob + n * 18].reshape(1, n, 3, 6).expand(count, -1, -1, -1)))
        o, ob = o + count * n * 3 * m, ob + n * 18
    done = [None] * len(parts)
    for slot, c in enumerate(cfgs):
        mine = [k for k, p in enumerate(parts) if p[0] == slot]
        if mine:
            r = _solve64(c, torch.cat([parts[k][1] for k in mine]), torch.cat([parts[k][2] for k in mine]),
                         case["iters"], None, None)
            counts = [parts[k][1].shape[0] for k in mine]
            for k, v in zip(mine, zip(*(t.split(counts) for t in r))):
                done[k] = v
    return [torch.cat([d[0].flatten() for d in done]), torch.cat([d[1].flatten() for d in done])] + \
        ([torch.cat([d[2] for d in done])] if case["resid"] else [])
