"""Single-flow defects on both sides of the tile rule (512-thread tiles up to two
tiles per compute unit, four at K = 1 with FP8 rows; 256-thread tiles above): the
last grid of the one and the first of the other, one patch wider, for every
input form: implicit Euler and Crank-Nicolson, the standard and the paper's
input, FP32, BF16 and FP8 rows; and the one-launch step (one tile per compute
unit).  At least two steps, so that the second takes the stored
corrected velocity, against the oracle.

Bounds: the step's own on rel-L2 (1e-5 with FP32 operands, 2e-2 with BF16; FP8
2e-2 on the per-patch output and 5e-3 on the state), on max-rel too for the
standard input.  The paper's input is not normalised, which leaves its largest
entries no such bound: there each 64 patches, in order, are within 0.25 of the
oracle on rel-L2 (a tile that is left out, or holds other rows, is off by about
its norm)."""
import numpy as np
import pytest

import oracle
from gpu_common import GpuRunner, assert_step_errors, merge_worst, rel_l2, step_errors
from paper_2008_11520_amd import synth

pytestmark = pytest.mark.gpu

# (K, precision, H, Crank-Nicolson, paper input)
FORMS = [(2, "fp32", 32, 0, 0), (2, "bf16", 32, 1, 0), (2, "fp32", 32, 1, 0), (2, "fp8", 64, 1, 0), (2, "fp8", 64, 0, 0),
         (2, "bf16", 96, 0, 1), (2, "fp32", 96, 0, 1), (2, "bf16", 96, 1, 1), (2, "fp32", 32, 1, 1),
         (3, "bf16", 64, 0, 0), (3, "fp32", 32, 0, 0), (3, "bf16", 64, 1, 0), (3, "fp32", 32, 1, 0), (3, "fp8", 64, 1, 0),
         (3, "bf16", 32, 0, 1), (3, "fp32", 32, 0, 1),
         (3, "bf16", 32, 1, 1), (3, "fp32", 32, 1, 1), (1, "fp8", 64, 0, 0), (1, "fp8", 64, 1, 0)]


def grid(K, wider, per_cu):
    """A grid of exactly per_cu tiles per compute unit, or one patch wider."""
    import torch
    tiles = torch.cuda.get_device_properties(0).multi_processor_count * per_cu
    side = 32 >> K                       # patches of a tile in each direction
    rows = 1
    while 4 * rows * rows <= tiles and tiles % (2 * rows) == 0:
        rows *= 2
    return side * (tiles // rows) + wider, side * rows


@pytest.mark.parametrize("wider", [0, 1])
@pytest.mark.parametrize("K,prec,H,cn,paper", FORMS)
def test_defect_rule_against_oracle(K, prec, H, cn, paper, wider):
    import paper_2008_11520_amd as pam
    nu = 1e-3
    nx, ny = grid(K, wider, 4 if K == 1 else 2)
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    w = synth.paper_net_weights(K, H, 1234) if paper else synth.xavier_weights(K, H, 0, 1234)
    flags = (pam.DNNMG_F_CRANK_NICOLSON if cn else 0) | (pam.DNNMG_F_PAPER_NET if paper else 0)
    g = GpuRunner(pam.DnnMG(pam.make_config(nx, ny, K, H, 0, flow.dt, nu, prec, flow.dirichlet, flags), flow.cxy, w))
    o = oracle.OracleFlow(nx, ny, K, H, 0, flow.dt, nu, flow.dirichlet, flow.cxy, w.astype(np.float64),
                          fp8=prec == "fp8", theta=0.5 if cn else 1.0, form=paper)
    worst = {}
    for n in range(2):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v, p, want=("Dbar", "bL", "dpatch"))
        e = step_errors(got, ref, o.h, nx, ny, K, flow.dirichlet)
        if prec == "fp8":
            assert e["Dbar_dirichlet_nonzero"] == 0 and e["dpatch"] < 2e-2 and e["h"] < 5e-3, (n, e)
            continue
        if paper:
            for k, r in (("dpatch", ref["dpatch"]), ("h", o.h)):
                for t in range(0, nx * ny, 64):
                    assert rel_l2(got[k][t:t + 64], r[t:t + 64]) < 0.25, (n, k, t)
            for k in ("h_max", "dpatch_max", "Dbar_max", "Dbar_edge_max"):
                e[k] = 0.0
        merge_worst(worst, e)
    if prec != "fp8":
        tol = 1e-5 if prec == "fp32" else 2e-2
        assert_step_errors(worst, tol, tol)
    g.g.close()


@pytest.mark.parametrize("wider", [0, 1])
@pytest.mark.parametrize("Hm", [0, 64])
def test_one_launch_rule_against_oracle(Hm, wider):
    import paper_2008_11520_amd as pam
    K, H, nu = 2, 64, 1e-3
    nx, ny = grid(K, wider, 1)
    flow = synth.channel_flow(nx, ny, 3, 0.005, perturb_seed=5)
    w = synth.xavier_weights(K, H, Hm, 1234)
    g = GpuRunner(pam.DnnMG(pam.make_config(nx, ny, K, H, Hm, flow.dt, nu, "bf16", flow.dirichlet), flow.cxy, w))
    o = oracle.OracleFlow(nx, ny, K, H, Hm, flow.dt, nu, flow.dirichlet, flow.cxy, w.astype(np.float64))
    worst = {}
    for n in range(3):
        v, p = flow.fields(n)
        got = g.step(v, p)
        ref = o.step(v, p, want=("Dbar", "bL"))
        merge_worst(worst, step_errors(got, ref, o.h, nx, ny, K, flow.dirichlet))
    assert_step_errors(worst, 2e-2, 2e-2)
    g.g.close()
