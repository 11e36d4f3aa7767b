"""Loading bodies far apart: the near-pair search costs what the bodies' own
triangles cost, whatever the empty space between them, and finds the same
pairs (those of each body, shifted)."""
import os
import time

import numpy as np
import pytest

from oracle import mesh as om
from paper_2111_11058_amd import cbfm
from synth import meshes

pytestmark = pytest.mark.skipif(not os.path.exists(cbfm.LIB_PATH), reason="libcbfm.so is not built")


def _bodies(V, T, offsets):
    return (np.concatenate([V + np.asarray(o, float) for o in offsets]),
            np.ascontiguousarray(np.concatenate([T + k * len(V) for k in range(len(offsets))]), np.int32))


def _best(V, T):
    best = np.inf
    for _ in range(3):
        t = time.perf_counter()
        cbfm.mesh_analyze(V, T)
        best = min(best, time.perf_counter() - t)
    return best


def test_time_does_not_grow_with_the_distance():
    V, T = meshes.geodesic(24, 1.0)
    near = _best(*_bodies(V, T, [(0, 0, 0), (3, 0, 0)]))
    for d in (30, 100, 10000):
        far = _best(*_bodies(V, T, [(0, 0, 0), (d, d, d)]))
        print(len(T), d, near, far)
        # sorting instead of counting the triangles, and nothing quadratic in a body
        assert far < 2.5 * near


@pytest.mark.parametrize("offsets", [
    [(0, 0, 0), (1000, 1000, 1000)],
    [(0, 0, 0), (1.05, 0, 0), (4e5, -3e5, 2e5), (4e5 + 1.05, -3e5, 2e5)],   # two touching pairs
    [(37.0 * k, -91.0 * k, 53.0 * k) for k in range(12)],
    [(0, 0, 0), (0, 0, 5000), (0, 0, -5000)],
    [(0, 0, 0), (5000, 0, 0), (0, 1.02, 0), (0, 0, -70)],
])
def test_pairs_of_scattered_bodies(offsets):
    V, T = meshes.icosphere(1, 0.5)
    V, T = _bodies(np.round(V * 2 ** 24) / 2 ** 24, T, offsets)
    near = cbfm.mesh_analyze(V, T)[3]
    m = om.build(V, T)
    assert np.array_equal(near[:, :2], om.near_pairs(m))
    assert np.array_equal(near[:, 2] != 0, [p == q or om.coplanar(m, p, q) for p, q in near[:, :2]])
