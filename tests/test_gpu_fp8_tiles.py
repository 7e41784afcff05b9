"""The persistent FP8 kernel at the edges of its 32-patch tiles: one patch less
and more than a tile, a 64-patch row tile whose second half is empty or holds
one patch, and grids on which a workgroup takes a second tile (32 x 1024
patches at H = 64, 32 x 256 at K = 3 and H = 128).  Reference: the oracle's
FP8 step; bounds: that step's own, 2e-2 relative L2 on the per-patch output
and 5e-3 on the state (both derived for means over tens of patches, so no
grid here has fewer than 31)."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, make_gpu_flow, rel_l2
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu

SMALL = [(31, 1), (8, 4), (11, 3), (13, 5), (43, 6)]
FORMS = [(1, 64, 0), (1, 128, 128), (2, 64, 64), (2, 128, 0), (2, 128, 128), (3, 64, 64), (3, 128, 128)]
CASES = [(nx, ny, *f) for nx, ny in SMALL for f in FORMS] + [(257, 131, 1, 64, 0), (91, 91, 3, 128, 128)]


@pytest.mark.parametrize("nx,ny,K,H,Hm", CASES)
def test_fp8_tiles_against_oracle(nx, ny, K, H, Hm):
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    w = synth.xavier_weights(K, H, Hm, 1234)
    g = GpuRunner(make_gpu_flow(flow, K, H, Hm, 1e-3, w, "fp8"))
    o = oracle.OracleFlow(nx, ny, K, H, Hm, flow.dt, 1e-3, flow.dirichlet, flow.cxy, w.astype(np.float64), fp8=True)
    for n in range(2):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v, p, want=("dpatch",))
        assert rel_l2(got["dpatch"], ref["dpatch"]) < 2e-2, n
        assert rel_l2(got["h"], o.h) < 5e-3, n
    g.g.close()
