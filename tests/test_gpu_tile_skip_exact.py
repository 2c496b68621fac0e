"""Time tiles that the MFMA forward kernel leaves out hold residuals that are exactly zero: a run of many iterations
equals as many runs of one iteration, which evaluate every tile, bit for bit.

The swarms are such that tiles are left out and come due again: robots that start apart in height and, by a large
penalty weight, sink slowly into crossing paths, and robots that separate from a crowd.  A model of the rule on the
run's own iterates shows it: how far the robots may have moved since a tile's last evaluation against half the least
separation found there."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

A, B, SKIN = 0.3, 0.4, 0.1     # safety semi-axes, margin of the pair lists as a fraction of them
K = 160

# robots, degree, horizon, weight of the collision rows: one and two robot tiles, one and more tiles per wave
SINKING = [(8, 10, 101, 40.0), (13, 13, 60, 25.0), (18, 9, 129, 30.0)]
CROWD = [(8, 10, 101, 1.2), (20, 11, 100, 1.2)]


def _case(n, degree, H, rho, sinking):
    cfg = W.SwarmConfig(n_robots=n, dims=3, degree=degree, horizon=H, t_final=8.0, safety_a=A, safety_b=B, vmax=60.0,
                        amax=60.0, rho_coll=rho, rho_vel=0.8, rho_acc=0.7)
    half = (1.4, 1.4, 0.3) if n <= 8 else (2.0, 2.0, 0.5)
    p = W.box_problem(cfg, 4, 0.15, seed=5 * n + degree, box=(tuple(-h for h in half), half), min_sep=0.45)
    x0 = p.xi_bar.copy()
    if sinking:
        x0[:, :, 2, 3:-3] += 0.9 * np.arange(n)[None, :, None]     # each robot at a height of its own
    return cfg, p, x0


def _left_out(cfg, states):
    """States [K, S, n, 3, m] of the iterations: the share of (iteration, sample, tile) that the rule leaves out, and
    the least scaled separation among those."""
    import paper_2501_19042_amd as P
    basis = torch.tensor(P.factor_table(cfg)["basis"][0]).cuda()
    n, H = cfg.n_robots, cfg.horizon
    i, j = np.triu_indices(n, 1)
    near = []
    for x in states:
        pos = torch.matmul(x.double(), basis.T)
        r = pos[:, i] - pos[:, j]
        s = ((r[:, :, 0] ** 2 + r[:, :, 1] ** 2) / A ** 2 + r[:, :, 2] ** 2 / B ** 2).amin(1)     # [S, H]
        near.append(torch.stack([s[:, t:t + 16].amin(1) for t in range(0, H, 16)], 1).sqrt())
    near = torch.stack(near).cpu().numpy()                          # [K, S, tiles]
    step = (states[1:] - states[:-1]).double().abs().amax(-1)       # [K - 1, S, n, 3]
    norm = step.norm(dim=-1).amax(-1).cpu().numpy()
    step = step.cpu().numpy()
    left = np.zeros_like(near, dtype=bool)
    lim = SKIN * np.array([A, A, B])
    for s in range(near.shape[1]):
        moved, drift, due = np.zeros((n, 3)), 0.0, np.full(near.shape[2], -1.0)
        for k in range(near.shape[0]):
            if k:
                moved, drift = moved + step[k - 1, s], drift + norm[k - 1, s]
            if k < 2 or (moved > lim).any():
                moved, drift, due[:] = np.zeros((n, 3)), 0.0, -1.0
            left[k, s] = drift <= due
            seen = ~left[k, s]
            due[seen] = np.where(near[k, s][seen] > 1, drift + 0.49 * ((near[k, s][seen] - 1) * min(A, B) - 1e-3), -1.0)
    return left.mean(), near[left].min()


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", [(*c, True) for c in SINKING] + [(*c, False) for c in CROWD])
def test_one_run_equals_single_iterations(shape, precision):
    import paper_2501_19042_amd as P
    cfg, p, x0 = _case(*shape)
    xb, bv, x = (torch.tensor(v, dtype=torch.float32).cuda() for v in (p.xi_bar, p.bvals, x0))
    sf = P.SafetyFilter([cfg])
    print(f"{shape} {precision}", flush=True)
    one = sf.project(xb, bv, K, precision=precision, xi0=x, ckpt_every=1)
    states, l = [], None
    for _ in range(K):
        states.append(x)
        step = sf.project(xb, bv, 1, precision=precision, xi0=x, lam0=l)
        x, l = step.xi, step.lam
    torch.cuda.synchronize()
    share, least = _left_out(cfg, torch.stack(states))
    print(f"{shape} {precision}: {share:.2f} of the tiles left out, least separation there {least:.4f}", flush=True)
    assert share >= 0.1 and least >= 1.0
    assert torch.equal(one.ckpt[:, 0].reshape(K, *xb.shape), torch.stack(states))
    assert torch.equal(one.xi, x) and torch.equal(one.lam, l)
