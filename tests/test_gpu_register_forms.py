"""Workspace solves in 16 bits on either side of the batch size at which the kernel's register budget changes (the
smaller batches hold their operands in registers, the larger re-read them): the samples of both agree bit for bit."""
from dataclasses import replace

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


# robots, degree, horizon: three and two coefficient steps of four, a ragged last time tile
@pytest.mark.parametrize("shape", [(13, 9, 75), (16, 10, 100), (9, 7, 33)])
@pytest.mark.parametrize("precision", ["bf16", "fp16"])
def test_budgets_agree(shape, precision):
    import paper_2501_19042_amd as P
    n, degree, H = shape
    cfg = W.SwarmConfig(n_robots=n, dims=3, degree=degree, horizon=H, t_final=8.0, safety_a=0.3, safety_b=0.4,
                        vmax=1.0, amax=1.0, rho_coll=1.2, rho_vel=0.8, rho_acc=0.7)
    half = (1.6, 1.6, 0.8)
    cfg = replace(cfg, ws_a=1.3 * half[0], ws_b=1.3 * half[2], rho_ws=0.9)
    p = W.box_problem(cfg, 8, 0.3, seed=3 * n, box=(tuple(-h for h in half), half), min_sep=0.35)
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    xb = torch.tensor(p.xi_bar, dtype=torch.float32).cuda()
    bv = torch.tensor(p.bvals, dtype=torch.float32).cuda()
    sf = P.SafetyFilter([cfg])
    got = {}
    for S in (4 * ncu - 1, 4 * ncu, 6 * ncu):   # 12 waves per CU: four samples of three; more take two waves or three
        out = sf.project(xb.repeat(-(-S // 8), 1, 1, 1)[:S].contiguous(), bv, 20, precision=precision)
        torch.cuda.synchronize()
        got[S] = out
        for name in ("xi", "lam", "resid"):
            print(f"{shape} {precision} S={S} {name}", flush=True)
            full = getattr(out, name)
            full = full[:S // 8 * 8].reshape(-1, 8, *full.shape[1:])
            assert all(torch.equal(full[0], q) for q in full), (S, name)
    a, b, c = got.values()
    for name in ("xi", "lam", "resid"):
        u, v, w = (getattr(t, name)[:8] for t in (a, b, c))
        assert torch.equal(u, v), name
        if name != "resid":   # other waves per sample: sums in another order, carried through the iterations
            assert ((w - u).abs().max() / u.abs().max()).item() <= 20 * 2.0 ** -16, name
