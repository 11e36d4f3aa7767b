"""Rounding of the regular fill: entries do not depend on where the body lies
(the points about a centroid and the centroids' offsets carry the rounding of
the triangle and of the pair, not of the coordinates), the float fill's error
over long distances averages over the quadrature points, and both precisions
agree with the oracle on either side of the centred phases' bounds."""
import dataclasses

import numpy as np
import pytest
import torch  # before the library, so that both use one runtime

pytestmark = pytest.mark.gpu


def _fill(w, prec):
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    mesh = cbfm.Mesh(w.V, w.T, w.edge_block, w.nblocks)
    med = cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r)
    out = torch.full((3, mesh.ne, mesh.ne), complex(np.nan, np.nan),
                     dtype=torch.complex128 if prec == cbfm.FP64 else torch.complex64, device="cuda")
    cbfm.fill_pmchwt(mesh, med, out, prec)
    return out.cpu().numpy().astype(np.complex128)


def _regular(w):
    """RWG pairs none of whose triangle pairs is near."""
    from paper_2111_11058_amd import cbfm
    E, TE, _, near = cbfm.mesh_analyze(w.V, w.T)
    A = np.zeros((len(w.T), len(E)))
    A[np.repeat(np.arange(len(w.T)), 3), TE.ravel()] = 1
    N = np.zeros((len(w.T), len(w.T)))
    N[near[:, 0], near[:, 1]] = 1
    return A.T @ N @ A == 0


@pytest.mark.parametrize("eps", [2.5, 2.5 - 0.5j, 30.0])
def test_place_of_the_body(eps):
    from paper_2111_11058_amd import cbfm
    from synth import configs
    w = dataclasses.replace(configs.small_cylinder(), eps_r=complex(eps))
    V = np.round(w.V * 2.0 ** 20) / 2.0 ** 20  # so that the shifted vertices are exact
    w = dataclasses.replace(w, V=V)
    far = dataclasses.replace(w, V=V + [4096.0, -2048.0, 8192.0])
    on = _regular(w)
    assert on.mean() > 0.3
    print("place", eps, flush=True)
    for x, r in zip(_fill(far, cbfm.FP64), _fill(w, cbfm.FP64)):
        # the same numbers to some tens of roundings; points rounded at 8192
        # would be off by 9e-13, 1e-11 of an edge
        e = np.linalg.norm((x - r)[on]) / np.linalg.norm(r[on])
        print(e)
        assert e < 1e-13


def test_float_over_long_distances():
    """Two bodies 50 wavelengths apart: per point pair the phase k R carries
    the roundings of a sum (halved by the root), the root and two products,
    0.5 x 2^-23 rms, which the weights average to 0.15 of it, 0.9e-8 k R.
    Roundings common to the pair (of the offset or its square) would come
    through whole, 1e-8 k R and more on top of that.  All relative to a
    triangle pair's charge term l_m l_n / (4 pi k R), of which an entry is
    the sum of four, two of either sign, that nearly cancel."""
    from paper_2111_11058_amd import cbfm
    from synth import configs, meshes
    V, T = meshes.icosphere(1, 0.17)
    d = np.array([31.3, 27.7, 26.9])
    V2, T2 = np.concatenate([V, V + d]), np.concatenate([T, T + len(V)])
    w = configs.sphere_c1()
    w = dataclasses.replace(w, V=V2, T=T2.astype(np.int32), edge_block=None, nblocks=1, eps_r=4.0 + 0j)
    print("float, long distances", flush=True)
    a, b = _fill(w, cbfm.FP64), _fill(w, cbfm.FP32)
    E = cbfm.mesh_analyze(V2, w.T)[0]
    one = E[:, 0] < len(V)
    ln, R = np.linalg.norm(V2[E[:, 0]] - V2[E[:, 1]], axis=1), np.linalg.norm(d)
    for o, k in ((1, 2 * np.pi), (2, 4 * np.pi)):
        x, r = b[o][np.ix_(one, ~one)], a[o][np.ix_(one, ~one)]
        four = 2.0 * np.outer(ln[one], ln[~one]) / (4 * np.pi * k * R)  # rms of four independent errors
        e = np.linalg.norm(x - r) / np.linalg.norm(four) / (k * R)
        print(o, e)
        assert e < 1.1e-8


@pytest.mark.parametrize("prec, tol", [("FP64", 1e-12), ("FP32", 2e-5)])
@pytest.mark.parametrize("scale, loss", [(0.98, 0.0), (1.02, 0.0), (0.9, 0.98), (0.9, 1.02), (2.0, 3.0)])
def test_centred_bounds(scale, loss, prec, tol):
    """The largest pair's phase span just below and above a sixth of a turn,
    its loss just below and above 1/24."""
    from oracle import fill, mesh as om
    from paper_2111_11058_amd import cbfm
    from synth import configs
    w = configs.small_cylinder()
    m = om.build(w.V, w.T)
    v = m.xyz - m.xyz.mean(axis=1, keepdims=True)
    most = 2 * 0.69614047802963365 * np.linalg.norm(v, axis=2).max()
    k0 = 2 * np.pi * scale / 6.0 / most / 3.0
    eps = (3.0 - 1j * loss / 24.0 / most / k0) ** 2
    k, _ = fill.media(k0, w.eta0, eps, 1.0)
    print("centred bounds", scale, loss, prec, flush=True)
    got = _fill(dataclasses.replace(w, k0=k0, eps_r=eps), getattr(cbfm, prec))
    for o, (x, r) in enumerate(zip(got, fill.fill_ops(m, k))):
        e = np.linalg.norm(x - r) / np.linalg.norm(r)
        print(o, e)
        assert e < tol
