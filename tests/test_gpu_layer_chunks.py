"""Equality-only QP layer at the edges of its chunking: one to many samples per chunk, more positions than
threads, sizes and pointers that rule out 16-byte accesses, in place; forward and reverse against the oracle's
closed form per robot-axis in FP64."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


# robots, dims, degree, samples, offset of the arrays in elements
@pytest.mark.parametrize("case", [(16, 3, 10, 1, 0), (16, 3, 10, 64, 0), (16, 3, 10, 64, 1), (2, 2, 5, 40000, 0),
                                  (3, 3, 6, 7000, 0), (32, 3, 14, 37, 0), (64, 3, 30, 3, 0), (33, 3, 20, 2000, 1)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_layer_chunks(case, prec):
    import paper_2501_19042_amd as P
    from paper_2501_19042_amd.sf import qp_equality, qp_equality_differentiable
    n, D, degree, S, off = case
    dt = torch.float64 if prec == "fp64" else torch.float32
    cfg = W.SwarmConfig(n_robots=n, dims=D, degree=degree, horizon=degree + 6, t_final=7.0, safety_a=0.3, safety_b=0.3,
                        vmax=1.0, amax=1.0)
    sf = P.SafetyFilter([cfg])
    m = degree + 1
    g = torch.Generator(device="cuda").manual_seed(n)

    def draw(shape):   # `off` elements into a larger buffer: not 16-byte aligned for off = 1
        num = int(np.prod(shape))
        return torch.randn(num + off, generator=g, device="cuda", dtype=torch.float64).to(dt)[off:].reshape(shape)

    x, go = draw((S, n, D, m)), draw((S, n, D, m))
    b = torch.randn((n, D, 6), generator=g, device="cuda", dtype=torch.float64).to(dt)
    bmap = torch.tensor(P.factor_table(cfg)["Bmap"]).cuda()
    at = [0, 1, 2, m - 3, m - 2, m - 1]
    want = x.double().clone()
    want[..., at] = torch.matmul(b.double(), bmap.T)
    xr, br = x.detach().requires_grad_(True), b.detach().requires_grad_(True)
    y = qp_equality_differentiable(sf, xr, br, precision=prec)
    gx, gb = torch.autograd.grad(y, (xr, br), go)
    eps = 1e-12 if prec == "fp64" else 2e-6
    assert ((y.double() - want).abs() <= eps * (1 + want.abs())).all()
    keep = go.clone()
    keep[..., at] = 0
    assert torch.equal(gx, keep)
    sums = go[..., at].double().sum(0)
    ref = torch.matmul(sums, bmap)
    # a sum of S terms of size one, rounded at every step: at most S units of rounding of its largest partial sum
    scale = torch.matmul(go[..., at].double().abs().sum(0), bmap.abs())
    unit = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    assert ((gb.double() - ref).abs() <= unit * (min(S, 64) + 12) * scale).all()
    z = x.clone()
    assert torch.equal(qp_equality(sf, z, b, precision=prec, out=z), y)
