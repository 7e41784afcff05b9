"""The neighbour tables of the library's unstructured meshes (the patch across
each edge and where its nodes lie, the corners' first gather-list entries, the
Dirichlet bits) against the meshes' gather lists, at every node of every patch.
CPU only."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2008_11520_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def _one_element():
    xy = np.array([[0.0, 0.0], [1.0, 0.0], [1.1, 1.0], [0.0, 0.9]])
    return synth.UMesh(xy, np.array([[0, 1, 2, 3]], np.int32), np.array([[1, 2]], np.int32), np.zeros((0, 3)),
                       np.zeros((0, 3), np.int32))


MESHES = {
    "one_element": _one_element,
    "cylinder_channel": lambda: synth.cylinder_channel_umesh(5),
    "shuffled_rotated": lambda: synth.structured_as_umesh(
        synth.perturb_interior(synth.rect_mesh(7, 5, 2.2, 0.41), 0.1, 3), synth.DIR_CHANNEL,
        order_seed=1, rotate_seed=2, renumber_seed=3)[0],
}


@pytest.fixture(scope="module")
def un(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("un") / "libun.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I",
                           os.path.join(ROOT, "paper_2008_11520_amd", "csrc"),
                           os.path.join(HERE, "umesh_neighbours_check.cpp"), "-o", so])
    return ctypes.CDLL(so)


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("K", [1, 2, 3])
def test_neighbour_tables_match_the_gather_lists(un, name, K):
    mesh = MESHES[name]()
    xy, el = np.ascontiguousarray(mesh.xy, np.float64), np.ascontiguousarray(mesh.elems, np.int32)
    dr, ci = np.ascontiguousarray(mesh.dirichlet_edges, np.int32), np.ascontiguousarray(mesh.circles, np.float64)
    cu = np.ascontiguousarray(mesh.curved, np.int32)
    vp = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    seen = ctypes.c_int()
    bad = un.un_check(xy.shape[0], el.shape[0], vp(xy), vp(el), dr.shape[0], vp(dr), ci.shape[0], vp(ci), cu.shape[0],
                      vp(cu), K, ctypes.byref(seen))
    assert bad == 0
    assert seen.value == el.shape[0] * ((1 << K) + 1) ** 2
