"""The regular fill's two phase forms (centred on the centroid distance for
pairs of small triangles, reduced per point pair otherwise) on both sides of
the bounds between them, and on a mesh whose wavefronts take either, against
the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

REV, EXP = 2.0 / 9.0, 1.0 / 16.0  # phase (revolutions) and loss bounds of the centred form
# Per entry at most 4 x 49 terms, each with a relative error of some tens of
# roundings (R, its reciprocal root, the phase k R of at most 40 radians
# rounded to 40 ulp, the moments): 1e-16 x 100 x sqrt(196), with a margin of 7.
TOL = 1e-12


@pytest.mark.parametrize("scale, loss, want", [
    (0.5, 0.0, "centred"), (0.99, 0.0, "centred"), (1.01, 0.0, "both"), (1.3, 0.0, "both"), (4.0, 0.0, "general"),
    (0.9, 0.99, "centred"), (0.9, 1.01, "both"), (0.9, 6.0, "general"),
])
def test_phase_forms(scale, loss, want):
    import torch
    from oracle import fill, mesh as om
    from paper_2111_11058_amd import cbfm
    from synth import configs
    w = configs.small_cylinder()
    m = om.build(w.V, w.T)
    v = m.xyz - m.xyz.mean(axis=1, keepdims=True)
    rad = 0.69614047802963365 * np.linalg.norm(v, axis=2).max(axis=1)  # the outermost quadrature point
    most, least = 2 * rad.max(), 2 * rad.min()
    # k2 = k0 (3 - j t), |Im k2| most = loss EXP, Re k2 most = scale REV turns
    k0 = 2 * np.pi * scale * REV / most / 3.0
    t = loss * EXP / most / k0
    eps = (3.0 - 1j * t) ** 2
    k, _ = fill.media(k0, w.eta0, eps, 1.0)
    span = lambda r: k[1].real * r / (2 * np.pi) > REV or -k[1].imag * r > EXP  # noqa: E731
    assert want == ("centred" if not span(most) else "general" if span(least) else "both")
    ref = fill.fill_ops(m, k)
    w = dataclasses.replace(w, k0=k0, eps_r=eps)
    mesh = cbfm.Mesh(w.V, w.T, w.edge_block, w.nblocks)
    med = cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r)
    out = torch.full((3, mesh.ne, mesh.ne), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
    print(f"fill phase form {want} scale {scale} loss {loss}", flush=True)
    cbfm.fill_pmchwt(mesh, med, out)
    for o, (x, r) in enumerate(zip(out.cpu().numpy(), ref)):
        err = np.linalg.norm(x - r) / np.linalg.norm(r)
        print(o, err)
        assert err < TOL, (o, err)
