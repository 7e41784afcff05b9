"""A mesh whose elements all meet in one node: its edges are found in a time that
does not depend on where that node comes in the numbering (each edge is listed
at the end with fewer elements), and the fine mesh is the reference
implementation's.  CPU only."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest

import oracle
from paper_2008_11520_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def fan(d, hub_first):
    """d quadrilaterals around the origin (hub, r_i, q_i, r_{i+1})."""
    i = np.arange(d)
    a = 2 * np.pi * i / d
    ring = np.stack([np.cos(a), np.sin(a)], 1)
    tips = 1.5 * np.stack([np.cos(a + np.pi / d), np.sin(a + np.pi / d)], 1)
    el = np.stack([np.full(d, 2 * d), i, d + i, (i + 1) % d], 1)
    xy = np.concatenate([ring, tips, np.zeros((1, 2))])
    if hub_first:
        xy, el = np.roll(xy, 1, axis=0), (el + 1) % (2 * d + 1)
    outer = np.stack([el[:, 1], el[:, 2]], 1)
    return synth.UMesh(np.ascontiguousarray(xy), np.ascontiguousarray(el, np.int32), outer.astype(np.int32),
                       np.zeros((0, 3)), np.zeros((0, 3), np.int32))


@pytest.fixture(scope="module")
def ub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("uh") / "libuh.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I",
                           os.path.join(ROOT, "paper_2008_11520_amd", "csrc"),
                           os.path.join(HERE, "umesh_build_check.cpp"), "-o", so])
    return ctypes.CDLL(so)


def _args(mesh):
    vp = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    return [mesh.xy.shape[0], mesh.elems.shape[0], vp(mesh.xy), vp(mesh.elems), mesh.dirichlet_edges.shape[0],
            vp(mesh.dirichlet_edges), 0, vp(mesh.circles), 0, vp(mesh.curved)]


def test_edges_of_a_hub_take_linear_time(ub):
    d, E, Fn = 20000, ctypes.c_int(), ctypes.c_int()
    took = {}
    for hub_first in (False, True):
        mesh = fan(d, hub_first)
        best = np.inf
        for _ in range(3):
            t = time.perf_counter()
            assert ub.ub_counts(*_args(mesh), 1, ctypes.byref(E), ctypes.byref(Fn)) == 0
            best = min(best, time.perf_counter() - t)
        assert (E.value, Fn.value) == (3 * d, 2 * d + 1 + 3 * d + d)
        took[hub_first] = best
    # (a walk over the hub's edges for each of them would take 8e8 steps, some fifty times the rest)
    assert took[True] < 4 * took[False] + 0.02, took


@pytest.mark.parametrize("hub_first", [False, True])
@pytest.mark.parametrize("K", [1, 2, 3])
def test_fan_matches_the_reference(ub, hub_first, K):
    mesh = fan(17, hub_first)
    ref = oracle.UFine(mesh, K)
    ne, n = 17, 1 << K
    nf, nc = (n + 1) ** 2, mesh.xy.shape[0]
    out = dict(pmap=np.empty((ne, nf), np.int32), fxy=np.empty((ref.Fn, 2)), rel=np.empty((ne, nf, 2)),
               mask=np.empty(ref.Fn, np.uint8), node_ptr=np.empty(ref.Fn + 1, np.int32),
               node_occ=np.empty(ne * nf, np.int32), cnode_ptr=np.empty(nc + 1, np.int32),
               cnode_occ=np.empty(4 * ne, np.int32), feat=np.empty((ne, 4), np.float32))
    vp = lambda x: x.ctypes.data_as(ctypes.c_void_p)
    assert ub.ub_build(*_args(mesh), K, *[vp(x) for x in out.values()]) == 0
    assert np.array_equal(out["pmap"], ref.pmap)
    assert np.array_equal(out["mask"].astype(bool), ref.mask)
    assert np.abs(out["fxy"] - ref.fxy).max() <= 1e-15 * np.abs(ref.fxy).max()
