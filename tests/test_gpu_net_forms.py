"""The network kernels at the edges of their tiles: one patch, one patch less
and more than a 64-row tile, and a mesh of several ragged tiles, for every
hidden size and operand type that a kernel is built for, with MLP widths
narrower and wider than the state, and the reset gate before and after U_h.
Reference: the FP64 oracle on the same inputs; bounds: the step's own, 1e-5
with FP32 operands and 2e-2 with BF16 operands."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, rel_l2, rel_max
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu

FORMS = [(1, 32, 0, 0), (1, 32, 32, 16), (1, 64, 64, 16), (2, 32, 64, 0), (2, 64, 64, 0), (2, 64, 256, 0),
         (2, 64, 0, 16), (2, 96, 96, 0), (2, 96, 32, 16), (2, 128, 64, 0), (2, 128, 128, 16), (3, 64, 64, 16)]


@pytest.mark.parametrize("nx,ny", [(1, 1), (9, 7), (8, 8), (13, 5), (43, 6)])
@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("bf16", 2e-2)])
def test_net_forms_against_oracle(nx, ny, prec, tol):
    import paper_2008_11520_amd as pam
    nu = 1e-3
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    for K, H, Hm, flags in FORMS:
        w = synth.xavier_weights(K, H, Hm, 1234)
        # (DNNMG_F_UNFUSED: the network kernel on its own, where the step would be one launch)
        cfg = pam.make_config(nx, ny, K, H, Hm, flow.dt, nu, prec, flow.dirichlet, flags | pam.DNNMG_F_UNFUSED)
        g = GpuRunner(pam.DnnMG(cfg, flow.cxy, w))
        o = oracle.OracleFlow(nx, ny, K, H, Hm, flow.dt, nu, flow.dirichlet, flow.cxy, w.astype(np.float64),
                              reset_after=bool(flags & pam.DNNMG_F_GRU_RESET_AFTER))
        for n in range(2):
            v, p = flow.fields(n)
            got = g.step(v, p)
            ref = o.step(v.astype(np.float64), p.astype(np.float64), want=("dpatch",))
            for k, r in (("dpatch", ref["dpatch"]), ("h", o.h)):
                a = got[k].reshape(np.asarray(r).shape)
                assert rel_l2(a, r) < tol and rel_max(a, r) < tol, (K, H, Hm, flags, nx, ny, n, k)
        g.g.close()
