"""An unstructured mesh with coarse nodes that no element uses (the first, two
neighbouring inner ones and the last in the numbering): the step writes every
entry of d and of the stored corrected velocity, zero and the coarse velocity at
such nodes, and reports nothing non-finite.  Reference: the oracle, whose mean
over no patch is zero; bounds: the step's own, 1e-5 with FP32 operands."""
import numpy as np
import pytest

import oracle
from paper_2008_11520_amd import synth

from gpu_common import rel_l2, rel_max, to_dev

pytestmark = pytest.mark.gpu


def with_lone_nodes(mesh, at):
    """The mesh with an unused node put before each node number in `at` (ascending)."""
    nc = mesh.xy.shape[0]
    new = np.array([i + sum(a <= i for a in at) for i in range(nc)], np.int32)
    lone = np.array([a + k for k, a in enumerate(at)])
    xy = np.full((nc + len(at), 2), 0.05)
    xy[new] = mesh.xy
    curved = mesh.curved.copy()
    curved[:, :2] = new[curved[:, :2]]
    return synth.UMesh(xy, new[mesh.elems], new[mesh.dirichlet_edges], mesh.circles, curved), lone


@pytest.mark.parametrize("K,H,Hm", [(1, 32, 0), (2, 64, 64), (3, 64, 0)])
def test_nodes_in_no_element(K, H, Hm):
    import torch
    import paper_2008_11520_amd as pam
    base = synth.cylinder_channel_umesh(4)
    nc = base.xy.shape[0]
    mesh, lone = with_lone_nodes(base, [0, nc // 2, nc // 2, nc])
    ff = synth.FourierField(synth.CHANNEL_LX, synth.CHANNEL_LY, 3).calibrate(mesh.xy)
    flow = synth.UFlow(mesh, 0.005, ff, inflow_max=1.5)
    w = synth.xavier_weights(K, H, Hm, 1234)
    g = pam.UDnnMG(K, H, Hm, flow.dt, 1e-3, mesh, w, "fp32", flags=pam.DNNMG_F_NANCHECK)
    o = oracle.OracleUFlow(mesh, K, H, Hm, flow.dt, 1e-3, w.astype(np.float64))
    d = torch.empty(2 * g.s["Fn"], device="cuda")
    u = torch.empty(2 * g.s["Fn"], device="cuda")
    b = torch.empty(2 * g.s["Nc"], dtype=torch.float64, device="cuda")
    for n in range(2):
        v, p = flow.fields(n)
        d.fill_(7.0)
        g.step(to_dev(v.reshape(-1)), to_dev(p), d)
        g.restrict_rhs(b)
        g.get_state(None, u)
        torch.cuda.synchronize()
        ref = o.step(v, p, want=("Dbar", "bL"))
        D, U = d.cpu().numpy().reshape(-1, 2), u.cpu().numpy().reshape(-1, 2)
        assert np.all(D[lone] == 0.0), n
        assert np.array_equal(U[lone], v[lone]), n
        assert rel_l2(D, ref["Dbar"]) < 1e-5 and rel_max(D, ref["Dbar"]) < 1e-5, n
        assert rel_max(b.cpu().numpy().reshape(-1, 2), ref["bL"]) < 1e-5, n
        assert g.nonfinite() == 0, n
    g.close()
