"""The right-hand side on both sides of its tile rule (16 x 16 fine elements up to
128 tiles of 32 x 32 at K <= 2 and 32 at K = 3): the last grid of the small tiles
and the first of the large ones, one patch wider.  The stage, implicit Euler and
Crank-Nicolson, against the oracle in FP64 (bound 1e-10: the order of the sums
alone differs); the step's averaged correction, state and b_L in FP32 (the
step's bound, 1e-5)."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, assert_step_errors, make_gpu_flow, merge_worst, rel_max, step_errors, to_dev
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu

GRIDS = [(1, 256, 128), (1, 257, 128), (2, 128, 64), (2, 129, 64), (3, 32, 16), (3, 33, 16)]


@pytest.mark.parametrize("K,nx,ny", GRIDS)
@pytest.mark.parametrize("cn", [False, True])
def test_rhs_few_stage_against_oracle(K, nx, ny, cn):
    import torch
    import paper_2008_11520_amd as pam
    H, nu = 32, 1e-3
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=7)
    w = synth.xavier_weights(K, H, 0, 1234)
    cfg = pam.make_config(nx, ny, K, H, 0, flow.dt, nu, "fp32", flow.dirichlet, pam.DNNMG_F_CRANK_NICOLSON if cn else 0)
    g = pam.DnnMG(cfg, flow.cxy, w)
    v, _ = flow.fields(1)
    dbar = (0.3 * synth.SplitMix64(5).uniform(2 * g.s["Fn"], -1.0, 1.0)).astype(np.float32)
    b = torch.empty(2 * g.s["Nc"], dtype=torch.float64, device="cuda")
    g.rhs_restrict(to_dev(v.reshape(-1)), to_dev(dbar), b)
    torch.cuda.synchronize()
    args = (nx, ny, K, flow.cxy.reshape(-1, 2), v.astype(np.float64), dbar.astype(np.float64).reshape(-1, 2), flow.dt)
    ref = oracle.rhs_restrict_theta(*args, nu, 0.5) if cn else oracle.rhs_restrict(*args)
    assert rel_max(b.cpu().numpy().reshape(-1, 2), ref) < 1e-10
    g.close()


@pytest.mark.parametrize("K,nx,ny", GRIDS)
def test_rhs_few_step_against_oracle(K, nx, ny):
    H, nu = 32, 1e-3
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=7)
    w = synth.xavier_weights(K, H, 0, 1234)
    g = GpuRunner(make_gpu_flow(flow, K, H, 0, nu, w, "fp32"))
    o = oracle.OracleFlow(nx, ny, K, H, 0, flow.dt, nu, flow.dirichlet, flow.cxy, w.astype(np.float64))
    worst = {}
    for n in range(2):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v.astype(np.float64), p.astype(np.float64), want=("Dbar", "bL", "dpatch"))
        merge_worst(worst, step_errors(got, ref, o.h, nx, ny, K, flow.dirichlet))
    assert_step_errors(worst, 1e-5, 1e-5)
    g.g.close()
