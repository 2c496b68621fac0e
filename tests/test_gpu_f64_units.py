"""FP64 solves in other units of length: the same problem scaled by a factor has the same solution scaled by it, and
the matrix-core kernel (whose drift bounds are kept in fp32) agrees with the kernel that evaluates every pair and ball
(generic=True)."""
from dataclasses import replace

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("unit", [1e-30, 1e-22, 1e-14, 1e-11, 1e-6, 1e6, 1e17, 1e25])
def test_scaled_problem(unit):
    from paper_2501_19042_amd import SafetyFilter
    cfg = W.SwarmConfig(n_robots=6, dims=3, degree=9, horizon=40, t_final=6.0, safety_a=0.3, safety_b=0.5, vmax=1.0,
                        amax=1.0, rho_coll=1.3, rho_vel=0.7, rho_acc=0.9, ws_a=1.6, ws_b=0.9, rho_ws=0.8, ws_x=0.1)
    p = W.box_problem(cfg, 3, 0.4, seed=5, box=((-1.2, -1.2, -0.6), (1.2, 1.2, 0.6)), min_sep=0.3)
    got = {}
    for u in (1.0, unit):
        c = replace(cfg, **{k: getattr(cfg, k) * u for k in ("safety_a", "safety_b", "vmax", "amax", "ws_a", "ws_b", "ws_x")})
        xb, bv = torch.tensor(p.xi_bar).cuda() * u, torch.tensor(p.bvals).cuda() * u
        sf = SafetyFilter([c])
        got[u] = [sf.project(xb, bv, 40, precision="fp64", generic=g) for g in (False, True)]
    torch.cuda.synchronize()
    ref = got[1.0][1]
    for out in got[unit]:
        for name in ("xi", "lam"):
            err = (getattr(out, name) / unit - getattr(ref, name)).abs().max().item()
            print(f"unit {unit:g} {name}: {err:.2e}", flush=True)
            assert err <= 1e-9 * (1 + getattr(ref, name).abs().max().item()), (unit, name, err)
