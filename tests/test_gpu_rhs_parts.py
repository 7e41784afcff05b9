"""The right-hand side at K = 3, where four lanes share a patch's node rows, at
the edges of its tiles of 4 x 4 patches, implicit Euler and Crank-Nicolson:
b_L against the oracle, FP64 on both sides (bound 1e-10: a sum of 81 products
in either order, rounded at 1e-16)."""
import numpy as np
import pytest

import oracle
from gpu_common import rel_max, to_dev
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (4, 4), (5, 4), (3, 9), (13, 5)])
@pytest.mark.parametrize("cn", [False, True])
def test_rhs_parts_against_oracle(nx, ny, cn):
    import torch
    import paper_2008_11520_amd as pam
    K, H, nu = 3, 32, 1e-3
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
