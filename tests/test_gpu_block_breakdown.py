"""Block GMRES with a single right-hand side whose Krylov space closes
exactly: with the tested field the first unit vector and Z_r diagonal, the
block A q - q (q^H A q) is zero to the last bit.  The first iteration solves
the system; the zero vector must not be divided by its norm."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("diag", [(1.0, 1.0), (2.0, 3.0), (-0.75, 5.0)])
def test_zero_block(diag):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    from synth import configs, meshes
    V, T = meshes.cube(3, 1.0)
    V = V - [0, 0, V[:, 2].max()]  # the upper face at z = 0: a wave along -z has phase 0 there
    inc = np.array([[0, 0, -1, 1, 0, 0.0]])
    mesh = cbfm.Mesh(V, T)
    med = cbfm.Medium.make(2 * np.pi, configs.ETA0, 2.5)
    v = torch.zeros((1, 2 * mesh.ne), dtype=torch.complex128, device="cuda")
    cbfm.rhs(mesh, med, inc, v)
    v = v.cpu().numpy()[0, :mesh.ne]
    # RWGs whose tested field is real and has a reciprocal that multiplies it back to 1
    hit = [e for e in range(mesh.ne) if v[e].imag == 0 and abs(v[e].real) > 1e-3 and v[e].real * (1.0 / v[e].real) == 1.0]
    assert len(hit) >= 3
    for e in hit[:3]:
        CJ = np.zeros((mesh.ne, 1), complex)
        CJ[e, 0] = 1.0 / v[e].real
        h = cbfm.cbf_import(mesh, [np.zeros((mesh.ne, 1), complex)], [CJ], [np.ones(1)])
        Zr = torch.tensor(np.diag(diag).astype(complex), device="cuda")
        o = cbfm.solve(mesh, med, h, Zr, inc, tol=1e-10, max_iter=8, restart=4, use_cmp=False, block=1)
        print("zero block", diag, e, o, flush=True)
        assert o["status"] == "OK" and o["relres"][0] <= 1e-15


@pytest.mark.parametrize("diag", [(1.0, 1.0), (2.0, 3.0)])
def test_rounding_block(diag):
    """The same with tested fields of any phase: the block is rounding, which
    the first pass may take for a direction and the second projects to zero."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from oracle import excitation, mesh as om
    from paper_2111_11058_amd import cbfm
    from synth import configs
    w = configs.sphere_c1()
    m = om.build(w.V, w.T)
    mesh = cbfm.Mesh(w.V, w.T)
    med = cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r)
    inc = configs.random_incidences(24, 5)
    CJ = excitation.rhs(m, inc, w.k0, w.eta0)[:m.ne, :1].copy()
    h = cbfm.cbf_import(mesh, [np.zeros((m.ne, 1), complex)], [CJ], [np.ones(1)])
    Zr = torch.tensor(np.diag(diag).astype(complex), device="cuda")
    print("rounding block", diag, flush=True)
    for q in range(len(inc)):
        o = cbfm.solve(mesh, med, h, Zr, inc[q:q + 1], tol=1e-10, max_iter=8, restart=4, use_cmp=False, block=1)
        assert o["status"] == "OK" and o["relres"][0] <= 1e-14, (q, o)
