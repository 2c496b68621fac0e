"""17 to 32 robots at degrees 5 to 7 (at most eight coefficients, two steps of four in the basis products) on the
matrix-core kernels: a batch of one shape, the same as a persistent launch, and gradients, against the oracle and the
FP64 reverse mode."""
from dataclasses import replace

import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

# robots, degree, horizon, samples, workspace: both ends of both ranges, a short last time tile, one tile in all
SHAPES = [(17, 5, 16, 3, False), (20, 7, 40, 3, True), (32, 6, 129, 2, False), (24, 7, 100, 300, False)]
BOUND = {"fp32": 1e-4, "bf16": 2e-3, "fp16": 2e-4}   # per sample, as for the other degrees


def _problem(n, degree, H, S, ws):
    cfg = W.SwarmConfig(n_robots=n, dims=3, degree=degree, horizon=H, t_final=8.0, safety_a=0.3, safety_b=0.4,
                        vmax=1.0, amax=1.0, rho_coll=1.2, rho_vel=0.8, rho_acc=0.7)
    half = (1.8, 1.8, 0.9)
    if ws:
        cfg = replace(cfg, ws_a=1.3 * half[0], ws_b=1.3 * half[2], rho_ws=0.9, ws_x=0.05, ws_y=-0.1, ws_z=0.02)
    return W.box_problem(cfg, S, 0.3, seed=11 * n + degree, box=(tuple(-h for h in half), half), min_sep=0.35)


@pytest.mark.parametrize("precision", list(BOUND))
@pytest.mark.parametrize("shape", SHAPES)
def test_solve_matches_oracle(shape, precision):
    from paper_2501_19042_amd import SafetyFilter
    p = _problem(*shape)
    sf = SafetyFilter([p.cfg])
    xb, bv = (torch.tensor(v, dtype=torch.float32).cuda() for v in (p.xi_bar, p.bvals))
    print(f"low degree {shape} {precision}", flush=True)
    one = sf.project(xb, bv, 25, precision=precision, want_status=True)
    per = sf.project(xb, bv, 25, precision=precision, persistent=True, want_status=True)
    torch.cuda.synchronize()
    k = min(3, xb.shape[0])
    rx, _, rr = O.sf_project(O.build_system(p.cfg), torch.tensor(p.xi_bar[:k]), torch.tensor(p.bvals), 25)
    for out in (one, per):
        err = (out.xi[:k].cpu().double() - rx).abs().flatten(1).amax(1) / rx.abs().flatten(1).amax(1)
        assert err.max().item() <= BOUND[precision], err
        assert torch.allclose(out.resid[:k].cpu().double(), rr, rtol=2e-2, atol=1e-5)


@pytest.mark.parametrize("shape", SHAPES[:3])
def test_gradients_match_fp64(shape):
    import paper_2501_19042_amd as P
    p = _problem(*shape)
    got = []
    for prec, dt in (("fp32", torch.float32), ("fp64", torch.float64)):
        xb, bv = (torch.tensor(v, dtype=torch.float32).to(dt).cuda() for v in (p.xi_bar, p.bvals))
        x0 = (xb * 1.01).requires_grad_(True)
        l0 = (0.05 * xb).requires_grad_(True)
        xb.requires_grad_(True)
        print(f"low degree gradients {shape} {prec}", flush=True)
        xi, lam, res, fpr = P.project_differentiable(P.SafetyFilter([p.cfg]), xb, bv, 10, xi0=x0, lam0=l0, ckpt_every=4,
                                                     precision=prec)
        loss = (fpr + res).sum() + ((xi - xb.detach()) ** 2).sum() + 0.1 * (lam * lam).sum()
        got.append(torch.autograd.grad(loss, (xb, x0, l0)))
    torch.cuda.synchronize()
    for name, a, b in zip(("xi_bar", "xi0", "lam0"), *got):
        # (degree 5 has no free coefficient: the gradient with respect to xi_bar is exactly zero)
        err, size = (a.double() - b).abs().max().item(), b.abs().max().item()
        assert err <= 2e-3 * size, (name, err, size)
