"""Edges and near pairs of meshes whose candidate grid is unusual (bodies far
apart, flat, tiny, shuffled numbering, the smallest closed mesh) against the
oracle's tables."""
import os

import numpy as np
import pytest

from oracle import mesh as om
from paper_2111_11058_amd import cbfm
from synth import meshes

pytestmark = pytest.mark.skipif(not os.path.exists(cbfm.LIB_PATH), reason="libcbfm.so is not built")


def _mesh(name):
    V, T = meshes.icosphere(1, 0.5)
    rng = np.random.default_rng(5)
    if name == "far":
        return np.concatenate([V, V + [900.0, -40.0, 3e4], V + [1.1, 0, 0]]), np.concatenate([T, T + len(V), T + 2 * len(V)])
    if name == "shuffled":
        p = rng.permutation(len(V))
        return V[p], np.argsort(p)[T][rng.permutation(len(T))]
    if name == "flat":
        V, T = meshes.cube(4, 1.0)
        return V * [1, 1, 1e-2], T
    if name == "tiny":
        return V * 1e-9, T
    if name == "uneven":  # one long body beside small triangles: a coarse grid
        V2, T2 = meshes.cube(1, 40.0)
        return np.concatenate([V, V2 + [0, 0, 60.0]]), np.concatenate([T, T2 + len(V)])
    return np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]), np.array([[0, 2, 1], [0, 1, 3], [0, 3, 2], [1, 2, 3]])


@pytest.mark.parametrize("name", ["far", "shuffled", "flat", "tiny", "uneven", "tetrahedron"])
def test_tables(name):
    V, T = _mesh(name)
    T = np.ascontiguousarray(T, np.int32)
    E, TE, TS, near = cbfm.mesh_analyze(V, T)
    m = om.build(V, T)
    assert np.array_equal(E, m.edges) and np.array_equal(TE, m.tri_edge) and np.array_equal(TS, m.tri_sign)
    assert np.array_equal(near[:, :2], om.near_pairs(m))
    assert np.array_equal(near[:, 2] != 0, [p == q or om.coplanar(m, p, q) for p, q in near[:, :2]])
