"""Batches that mix swarms of up to 16 and of more than 16 robots, degrees, horizons and workspaces.  One of more than
16 robots makes the reverse sweep, the FP64 solve and the feasibility check run the whole batch on two robot tiles; a
mix of 2D and 3D sends FP64 to the generic kernel.  Each problem agrees with a call of its own."""
from dataclasses import replace

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _problems(spec):
    out = []
    for k, (n, dims, degree, H, S, ws) in enumerate(spec):
        cfg = W.SwarmConfig(n_robots=n, dims=dims, degree=degree, horizon=H, t_final=8.0, safety_a=0.3, safety_b=0.4,
                            vmax=1.0, amax=1.0, rho_coll=1.2, rho_vel=0.8, rho_acc=0.7)
        half = (1.8, 1.8, 0.9)[:dims]
        if ws:
            cfg = replace(cfg, ws_a=2.2, ws_b=1.1, rho_ws=0.9, ws_x=0.05, ws_y=-0.1, ws_z=0.02)
        out.append(W.box_problem(cfg, S, 0.3, seed=40 + k, box=(tuple(-h for h in half), half), min_sep=0.3))
    return out


def _flat(probs, key, dt):
    return torch.cat([torch.tensor(getattr(p, key), dtype=torch.float32).to(dt).reshape(-1) for p in probs]).cuda()


def _each(probs, flat):
    o = 0
    for p in probs:
        num = p.xi_bar.size
        yield flat[o:o + num].reshape(p.xi_bar.shape)
        o += num


# robots, dims, degree, horizon, samples, workspace
LARGE = [(8, 3, 8, 40, 3, False), (24, 3, 11, 70, 2, True), (16, 3, 15, 100, 2, True), (19, 3, 6, 17, 3, False)]
PLANAR = [(5, 2, 10, 50, 3, False), (12, 3, 9, 40, 2, True), (20, 2, 8, 33, 2, False)]
BOTH = [(6, 2, 8, 40, 2, False), (10, 3, 9, 50, 2, True), (18, 3, 7, 20, 1, False)]


@pytest.mark.parametrize("want_resid", [True, False])
def test_reverse_mode(want_resid):
    import paper_2501_19042_amd as P
    probs = _problems(LARGE)
    batch = P.Batch([(k, p.xi_bar.shape[0]) for k, p in enumerate(probs)])
    sf = P.SafetyFilter([p.cfg for p in probs])

    def grads(f, xb, bv, b=None):
        x0, l0 = (xb * 1.02).requires_grad_(True), (0.05 * xb).requires_grad_(True)
        xb = xb.clone().requires_grad_(True)
        xi, lam, res, fpr = P.project_differentiable(f, xb, bv, 9, xi0=x0, lam0=l0, ckpt_every=4, batch=b)
        loss = fpr.sum() + ((xi - xb.detach()) ** 2).sum() + 0.1 * (lam * lam).sum()
        if want_resid:
            loss = loss + res.sum()
        return torch.autograd.grad(loss, (xb, x0, l0))

    print("mixed reverse", want_resid, flush=True)
    whole = grads(sf, _flat(probs, "xi_bar", torch.float32), _flat(probs, "bvals", torch.float32), batch)
    parts = [list(_each(probs, g)) for g in whole]
    for k, p in enumerate(probs):
        own = grads(P.SafetyFilter([p.cfg]), torch.tensor(p.xi_bar, dtype=torch.float32).cuda(),
                    torch.tensor(p.bvals, dtype=torch.float32).cuda())
        torch.cuda.synchronize()
        for name, a, b in zip(("xi_bar", "xi0", "lam0"), (q[k] for q in parts), own):
            # (both within the fp32 reverse mode's bound of the exact gradient)
            err = (a - b).abs().max().item()
            assert err <= 2e-3 * b.abs().max().item(), (k, name, err)


@pytest.mark.parametrize("spec", [LARGE, PLANAR, BOTH])
def test_fp64_solve_and_feasibility(spec):
    import paper_2501_19042_amd as P
    probs = _problems(spec)
    batch = P.Batch([(k, p.xi_bar.shape[0]) for k, p in enumerate(probs)])
    sf = P.SafetyFilter([p.cfg for p in probs])
    xb, bv = _flat(probs, "xi_bar", torch.float64), _flat(probs, "bvals", torch.float64)
    print("mixed fp64", spec, flush=True)
    out = sf.project(xb, bv, 25, batch=batch, precision="fp64", want_status=True)
    viol = sf.feasibility(out.xi, bv, batch=batch, precision="fp64")
    torch.cuda.synchronize()
    s = 0
    for p, xi, lam in zip(probs, _each(probs, out.xi), _each(probs, out.lam)):
        S = p.xi_bar.shape[0]
        f = P.SafetyFilter([p.cfg])
        x1 = torch.tensor(p.xi_bar, dtype=torch.float32).double().cuda()
        b1 = torch.tensor(p.bvals, dtype=torch.float32).double().cuda()
        own = f.project(x1, b1, 25, precision="fp64", generic=True, want_status=True)
        v = f.feasibility(own.xi, b1, precision="fp64")
        torch.cuda.synchronize()
        for name, a, b in (("xi", xi, own.xi), ("lam", lam, own.lam), ("resid", out.resid[s:s + S], own.resid),
                           ("violations", viol[s:s + S], v)):
            err = ((a - b).abs() / (1 + b.abs())).max().item()
            assert err <= 1e-9, (p.cfg.n_robots, name, err)
        assert torch.equal(out.status[s:s + S], own.status)
        s += S
