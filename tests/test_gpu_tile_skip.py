"""Time tiles that the MFMA forward kernel leaves out between contacts: one run of many iterations against as many
runs of one iteration, each of which evaluates every tile."""
from dataclasses import replace

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# robots, degree, horizon, samples, workspace: both robot tiles, one tile in all, several per wave, a short last one
SHAPES = [(2, 6, 16, 4, False), (8, 10, 101, 6, False), (16, 10, 100, 40, True), (16, 15, 256, 6, False),
          (17, 9, 33, 4, False), (32, 10, 128, 8, True)]
K = 96


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_run_equals_single_iterations(shape, precision):
    import paper_2501_19042_amd as P
    n, degree, H, S, ws = shape
    cfg = W.SwarmConfig(n_robots=n, dims=3, degree=degree, horizon=H, t_final=8.0, safety_a=0.3, safety_b=0.4,
                        vmax=1.0, amax=1.0, rho_coll=1.2, rho_vel=0.8, rho_acc=0.7)
    half = (1.6, 1.6, 0.8) if n > 8 else (1.0, 1.0, 0.4)
    if ws:
        cfg = replace(cfg, ws_a=1.3 * half[0], ws_b=1.3 * half[2], rho_ws=0.9)
    p = W.box_problem(cfg, S, 0.3, seed=5 * n + degree, box=(tuple(-h for h in half), half), min_sep=0.35)
    xb = torch.tensor(p.xi_bar, dtype=torch.float32).cuda()
    bv = torch.tensor(p.bvals, dtype=torch.float32).cuda()
    sf = P.SafetyFilter([cfg])
    one = sf.project(xb, bv, iters=K, precision=precision)
    x, l = None, None
    for _ in range(K):
        step = sf.project(xb, bv, iters=1, xi0=x, lam0=l, precision=precision)
        x, l = step.xi, step.lam
    torch.cuda.synchronize()
    # rounding of one iteration (about 32 terms in fp32; the 16-bit split keeps 16 or more bits of a position),
    # carried through K iterations of a nonexpansive map
    tol = K * (32 * 2.0 ** -24 if precision == "fp32" else 2.0 ** -16)
    for name, a, b in (("xi", one.xi, x), ("lam", one.lam, l)):
        err = ((a - b).abs().max() / b.abs().max()).item()
        print(f"{shape} {precision} {name}: {err:.2e}", flush=True)
        assert err <= tol, (name, err)
