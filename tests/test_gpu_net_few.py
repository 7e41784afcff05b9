"""The streamed network kernel on both sides of its tile rule (16 patches a
workgroup up to 8192 patches, 64 above; at H >= 96 in BF16 up to 4096, above
that the persistent kernels): the last count of the one and the first of the
other, whose last tile holds one patch.  Reference: the FP64 oracle; bounds: the
step's own, 1e-5 with FP32 operands and 2e-2 with BF16 operands."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, rel_l2, rel_max
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu

WIDE = [("fp32", 1, 32, 0, 0), ("fp32", 2, 64, 64, 0), ("fp32", 2, 96, 32, 16), ("bf16", 2, 64, 256, 0)]
HEAVY = [("bf16", 2, 96, 96, 0), ("bf16", 2, 128, 128, 0), ("bf16", 3, 128, 0, 0)]
CASES = [(nx, ny, *f) for nx, ny in ((128, 64), (2731, 3)) for f in WIDE]
CASES += [(nx, ny, *f) for nx, ny in ((64, 64), (241, 17), (9, 7)) for f in HEAVY]


@pytest.mark.parametrize("nx,ny,prec,K,H,Hm,flags", CASES)
def test_net_few_patches_against_oracle(nx, ny, prec, K, H, Hm, flags):
    import paper_2008_11520_amd as pam
    nu, tol = 1e-3, {"fp32": 1e-5, "bf16": 2e-2}[prec]
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    w = synth.xavier_weights(K, H, Hm, 1234)
    g = GpuRunner(pam.DnnMG(pam.make_config(nx, ny, K, H, Hm, flow.dt, nu, prec, flow.dirichlet, flags), flow.cxy, w))
    o = oracle.OracleFlow(nx, ny, K, H, Hm, flow.dt, nu, flow.dirichlet, flow.cxy, w.astype(np.float64),
                          reset_after=bool(flags & pam.DNNMG_F_GRU_RESET_AFTER))
    for n in range(2):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v.astype(np.float64), p.astype(np.float64), want=("dpatch",))
        for k, r in (("dpatch", ref["dpatch"]), ("h", o.h)):
            a = got[k].reshape(np.asarray(r).shape)
            assert rel_l2(a, r) < tol and rel_max(a, r) < tol, (n, k)
    g.g.close()
