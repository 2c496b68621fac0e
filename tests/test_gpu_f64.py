"""FP64 matrix-core kernel against the kernel that evaluates every pair and ball in every iteration
(generic=True), which the other tests hold to the oracle, and against the oracle itself."""
import numpy as np
import pytest
import torch
from dataclasses import replace

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _close(a, b, what):
    err = ((a - b).abs() / (1.0 + b.abs())).max().item()
    assert err <= 1e-9, f"{what}: {err:.3e}"


# robots, dims, degree, horizon, samples, workspace: both robot tiles and their edges, the smallest and
# largest polynomials, horizons of one tile, a one-step last tile and more tiles than waves; more samples
# than compute units take four waves per sample
SHAPES = [(2, 3, 5, 16, 2, False), (4, 2, 10, 100, 8, False), (16, 3, 10, 100, 3, False), (16, 3, 15, 256, 2, True),
          (17, 3, 12, 33, 2, False), (32, 3, 12, 120, 2, False), (9, 3, 7, 17, 300, True), (13, 2, 9, 129, 300, False),
          (31, 3, 15, 129, 1, True), (20, 2, 8, 64, 3, False)]


def _inputs(n, D, degree, H, S, ws):
    cfg = W.SwarmConfig(n_robots=n, dims=D, degree=degree, horizon=H, t_final=6.0, safety_a=0.3, safety_b=0.5,
                        vmax=1.5, amax=2.0, rho_coll=1.3, rho_vel=0.7, rho_acc=0.9)
    if ws:
        cfg = replace(cfg, ws_a=2.0, ws_b=1.1, rho_ws=0.8, ws_x=0.1, ws_y=-0.2, ws_z=0.05)
    half = np.array([1.6, 1.6, 0.9])[:D]
    p = W.box_problem(cfg, S, 0.4, seed=n + degree, box=(tuple(-half), tuple(half)), min_sep=0.35 if D == 3 else 0.3)
    g = torch.Generator().manual_seed(n)
    xb, bv = torch.tensor(p.xi_bar), torch.tensor(p.bvals)
    x0 = xb + 0.1 * torch.randn(xb.shape, generator=g, dtype=torch.float64)
    l0 = 0.05 * torch.randn(xb.shape, generator=g, dtype=torch.float64)
    return cfg, xb, bv, x0, l0


@pytest.mark.parametrize("shape", SHAPES)
def test_f64_matches_dense_kernel(shape):
    from paper_2501_19042_amd import SafetyFilter
    cfg, xb, bv, x0, l0 = _inputs(*shape)
    sf = SafetyFilter([cfg])
    kw = dict(precision="fp64", xi0=x0.cuda(), lam0=l0.cuda(), ckpt_every=7, fp_residual=True, want_status=True)
    a = sf.project(xb.cuda(), bv.cuda(), 30, **kw)
    b = sf.project(xb.cuda(), bv.cuda(), 30, generic=True, **kw)
    torch.cuda.synchronize()
    for name in ("xi", "lam", "resid", "ckpt"):
        _close(getattr(a, name), getattr(b, name), name)
    assert torch.equal(a.status, b.status)
    k = min(2, xb.shape[0])
    rx, rl, rr = O.sf_project(O.build_system(cfg), xb[:k], bv, 30, xi0=x0[:k], lam0=l0[:k])
    _close(a.xi[:k].cpu(), rx, "oracle xi")
    _close(a.resid[:k, :2].cpu(), rr, "oracle residual")


def test_f64_non_finite_inputs():
    """Without a status array, a NaN coefficient spreads as in the dense kernel and other samples stay."""
    from paper_2501_19042_amd import SafetyFilter
    cfg, xb, bv, x0, l0 = _inputs(6, 3, 9, 40, 3, True)
    xb[1, 2, 1, 4] = float("nan")
    sf = SafetyFilter([cfg])
    a = sf.project(xb.cuda(), bv.cuda(), 12, precision="fp64")
    b = sf.project(xb.cuda(), bv.cuda(), 12, precision="fp64", generic=True)
    torch.cuda.synchronize()
    for name in ("xi", "lam"):
        u, v = getattr(a, name), getattr(b, name)
        assert torch.equal(u.isnan(), v.isnan()) and bool(u[1].isnan().any()) and not bool(u[0].isnan().any())
        ok = ~v.isnan()
        _close(u[ok], v[ok], name)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_feasibility_matches_oracle(shape, prec):
    """Violations from the matrix-core check against the oracle's, also where nothing collides or all do."""
    from paper_2501_19042_amd import SafetyFilter
    cfg, xb, bv, x0, _ = _inputs(*shape)
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = x0.to(dt)[:40]
    x[0] *= 0.01      # every pair inside the safety distance
    v = SafetyFilter([cfg]).feasibility(x.cuda(), bv.to(dt).cuda(), precision=prec).cpu()
    _close(v, O.feasibility(O.build_system(cfg), x.double(), bv.to(dt).double()), "violations")
