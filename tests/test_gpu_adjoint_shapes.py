"""Matrix-core reverse mode (fp32) at the edges of its shapes against the FP64 reverse mode on the GPU, which
test_gpu_adjoint.py holds to autograd through the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# robots, degree, horizon, samples, iterations, checkpoint interval, workspace: both robot tiles and their
# edges, coefficient steps of 2 to 4, one and more time tiles per wave, a one-step last tile, segments that do
# not divide the iterations or exceed them, more samples than compute units, and a scratch of several groups
SHAPES = [(2, 6, 16, 2, 9, 4, False), (5, 7, 17, 3, 6, 20, True), (16, 15, 256, 2, 8, 3, False),
          (13, 10, 129, 2, 12, 5, True), (17, 9, 33, 2, 9, 9, False), (24, 11, 80, 2, 12, 5, True),
          (26, 15, 97, 1, 6, 4, False), (32, 12, 60, 3, 10, 1, True), (16, 10, 100, 300, 12, 5, False),
          (18, 8, 40, 1, 5, 2, False)]


@pytest.mark.parametrize("shape", SHAPES)
def test_mfma_adjoint_shapes(shape):
    import paper_2501_19042_amd as P
    n, degree, H, S, iters, every, ws = shape
    cfg = W.SwarmConfig(n_robots=n, dims=3, degree=degree, horizon=H, t_final=8.0, safety_a=0.3, safety_b=0.4,
                        vmax=1.0, amax=1.0, rho_coll=1.2, rho_vel=0.8, rho_acc=0.7)
    half = (1.6, 1.6, 0.8) if n > 8 else (1.0, 1.0, 0.4)
    if ws:
        cfg = replace(cfg, ws_a=1.3 * half[0], ws_b=1.3 * half[2], rho_ws=0.9, ws_x=0.05, ws_y=-0.1, ws_z=0.02)
    p = W.box_problem(cfg, min(S, 3), 0.3, seed=7 * n + degree, box=(tuple(-h for h in half), half), min_sep=0.35)
    rng = np.random.default_rng(n)
    reps = -(-S // p.xi_bar.shape[0])
    xi = p.xi_bar
    ins = {}
    for dt in (torch.float32, torch.float64):
        r = np.random.default_rng(n)
        vals = [xi, xi + 0.05 * r.normal(size=xi.shape), 0.1 * r.normal(size=xi.shape)]
        ins[dt] = [torch.tensor(v, dtype=torch.float32).repeat(reps if dt == torch.float32 else 1, 1, 1, 1)[:S]
                   .to(dt).cuda().requires_grad_(True) for v in vals]
    wr = torch.tensor(rng.uniform(0.5, 1.5, size=xi.shape[0]), dtype=torch.float32)
    got = {}
    for dt, prec in ((torch.float32, "fp32"), (torch.float64, "fp64")):
        sf = P.SafetyFilter([cfg])
        xb, x0, l0 = ins[dt]
        wt = wr.repeat(reps)[:xb.shape[0]].to(dt).cuda()
        xk, lk, res, fpr = P.project_differentiable(sf, xb, torch.tensor(p.bvals, dtype=dt).cuda(), iters, xi0=x0,
                                                    lam0=l0, ckpt_every=every, precision=prec)
        loss = 0.3 * (wt * fpr).sum() + ((xk - xb.detach()) ** 2).sum() + (wt * res).sum() + 0.1 * (lk * lk).sum()
        got[prec] = torch.autograd.grad(loss, (xb, x0, l0))
    torch.cuda.synchronize()
    k = got["fp64"][0].shape[0]
    for name, a, b in zip(("xi_bar", "xi0", "lam0"), got["fp32"], got["fp64"]):
        err = ((a[:k].double() - b).abs().max() / b.abs().max()).item()
        print(f"{shape} {name}: {err:.2e}", flush=True)
        assert err <= 2e-3, (name, err)
        for q in range(k, a.shape[0], k):   # repeated samples
            assert torch.equal(a[q:q + k], a[:a[q:q + k].shape[0]]), name
