"""The BF16 network kernel that keeps its weights in registers (H = 128, or
K = 3) at the edges of its tiles of 32 (K = 3) and 64 patches: one patch less
and more than a tile, a 64-patch row tile whose second half is empty, 256 row
tiles and 257, the last one of a single patch, so that a workgroup takes a
second tile.  The network's output and state against the FP64 oracle within the
step's bound for BF16 operands, 2e-2; and a batch of 261 row tiles against the
same flows stepped alone, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, make_gpu_flow, rel_l2, rel_max, to_dev
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(31, 1), (8, 4), (11, 3), (9, 7), (13, 5), (128, 128), (145, 113)])
@pytest.mark.parametrize("K,H,Hm", [(1, 128, 0), (2, 128, 128), (3, 64, 64), (3, 128, 0)])
def test_wide_tiles_against_oracle(nx, ny, K, H, Hm):
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    w = synth.xavier_weights(K, H, Hm, 1234)
    g = GpuRunner(make_gpu_flow(flow, K, H, Hm, 1e-3, w, "bf16"))
    o = oracle.OracleFlow(nx, ny, K, H, Hm, flow.dt, 1e-3, flow.dirichlet, flow.cxy, w.astype(np.float64))
    for n in range(2):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v.astype(np.float64), p.astype(np.float64), want=("dpatch",))
        for k, r in (("dpatch", ref["dpatch"]), ("h", o.h)):
            a = got[k].reshape(np.asarray(r).shape)
            assert rel_l2(a, r) < 2e-2 and rel_max(a, r) < 2e-2, (n, k)
    g.g.close()


@pytest.mark.parametrize("K,H,Hm", [(2, 128, 128), (3, 128, 0)])
def test_wide_tiles_batch_equals_single_flows(K, H, Hm):
    import torch
    import paper_2008_11520_amd as pam
    w = synth.xavier_weights(K, H, Hm, 5)
    # row tiles 1, 256, 3, 1
    flows = [synth.channel_flow(9, 7, 3, 0.005), synth.channel_flow(128, 128, 4, 0.005, perturb_seed=8),
             synth.unit_square_flow(13, 11, 2, 0.01), synth.channel_flow(5, 3, 9, 0.005)]
    single = [GpuRunner(make_gpu_flow(f, K, H, Hm, 1e-3, w, "bf16")) for f in flows]
    model = make_gpu_flow(flows[0], K, H, Hm, 1e-3, w, "bf16")
    batched = [make_gpu_flow(f, K, H, Hm, 1e-3, w, "bf16", share=model) for f in flows]
    runners = [GpuRunner(b) for b in batched]
    batch = pam.Batch(8)
    for n in range(2):
        fields = [f.fields(n) for f in flows]
        ref = [r.step(v, p) for r, (v, p) in zip(single, fields)]
        batch.step(batched, [to_dev(v.reshape(-1)) for v, _ in fields], [to_dev(p) for _, p in fields],
                   [r.dbar for r in runners])
        for r, b, rf in zip(runners, batched, ref):
            b.get_state(r.h, None)
            torch.cuda.synchronize()
            assert np.array_equal(r.dbar.cpu().numpy().reshape(-1, 2), rf["Dbar"])
            assert np.array_equal(r.h.cpu().numpy().reshape(b.s["P"], -1), rf["h"])
    batch.close()
    for x in batched + [model] + [r.g for r in single]:
        x.close()
