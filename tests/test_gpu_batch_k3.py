"""Batched steps at K = 3, whose defect and right-hand side take one tile per
block: from a graph whose membership grows past the grid it was captured with
(2048 tiles; the second flow alone has 2250), shrinks and returns, against
single-flow steps, bit for bit, on each operand type."""
import numpy as np
import pytest

from gpu_common import GpuRunner, make_gpu_flow, to_dev
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,H,Hm", [("fp32", 32, 0), ("bf16", 64, 64), ("fp8", 64, 0)])
def test_k3_graph_follows_membership_bitwise(prec, H, Hm):
    import torch
    import paper_2008_11520_amd as pam
    K = 3
    w = synth.xavier_weights(K, H, Hm, 5)
    flows = [synth.channel_flow(9, 7, 3, 0.005), synth.channel_flow(200, 180, 4, 0.005, perturb_seed=8),
             synth.unit_square_flow(1, 1, 2, 0.01)]
    single = [GpuRunner(make_gpu_flow(f, K, H, Hm, 1e-3, w, prec)) for f in flows]
    model = make_gpu_flow(flows[0], K, H, Hm, 1e-3, w, prec)
    ctxs = [make_gpu_flow(f, K, H, Hm, 1e-3, w, prec, share=model) for f in flows]
    runners = [GpuRunner(c) for c in ctxs]
    batch = pam.Batch(4)
    st = torch.cuda.Stream()
    nstep = [0] * len(flows)
    for members in ([0], [0, 2], [2, 1, 0], [2], [1, 0]):
        fields = {i: flows[i].fields(nstep[i]) for i in members}
        ref = {i: single[i].step(*fields[i]) for i in members}
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            vs = [to_dev(fields[i][0].reshape(-1)) for i in members]
            ps = [to_dev(fields[i][1]) for i in members]
            batch.prepare([ctxs[i] for i in members], vs, ps, [runners[i].dbar for i in members],
                          [runners[i].bL for i in members], stream=st)
            batch.launch(graph=True, stream=st)
        st.synchronize()
        for i in members:
            r, c = runners[i], ctxs[i]
            c.get_state(r.h, None)
            torch.cuda.synchronize()
            assert np.array_equal(r.dbar.cpu().numpy().reshape(-1, 2), ref[i]["Dbar"]), (members, i)
            assert np.array_equal(r.bL.cpu().numpy().reshape(-1, 2), ref[i]["bL"]), (members, i)
            assert np.array_equal(r.h.cpu().numpy().reshape(c.s["P"], -1), ref[i]["h"]), (members, i)
            nstep[i] += 1
    assert batch.captures == 2
    batch.close()
    for x in ctxs + [model] + [r.g for r in single]:
        x.close()
