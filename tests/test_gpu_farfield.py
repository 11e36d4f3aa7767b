"""RCS of given currents at the far-field kernel's edges: groups of four
right-hand sides (common directions) with remainders, one right-hand side a
block (monostatic), and the triangles in one chunk or many, against the
oracle's radiation integrals of the same currents."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name, nrhs, nd", [("c1", 1, 1), ("c1", 2, 73), ("c1", 4, 3), ("c1", 5, 1), ("c1", 9, 600),
                                            ("c1", 1, 0), ("c1", 6, 0), ("c3", 3, 2), ("c3", 7, 37), ("c3", 3, 0)])
def test_rcs_of_currents(name, nrhs, nd):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from oracle import excitation, mesh as om
    from paper_2111_11058_amd import cbfm
    from synth import configs
    w = configs.sphere_c1() if name == "c1" else configs.sphere_c3()
    m = om.build(w.V, w.T)
    mesh = cbfm.Mesh(w.V, w.T, w.edge_block, w.nblocks)
    med = cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r)
    sizes = np.bincount(w.edge_block, minlength=w.nblocks)
    C = [[configs.random_complex((int(s), 2), 50 * h + a) for a, s in enumerate(sizes)] for h in range(2)]
    h = cbfm.cbf_import(mesh, C[0], C[1], [np.ones(2) for _ in sizes])
    Zr = torch.eye(h.n_cbf, dtype=torch.complex128, device="cuda")
    inc = configs.random_incidences(nrhs, 3)
    dirs = configs.random_incidences(nd, 4)[:, :3].copy() if nd else None
    jt = torch.zeros((nrhs, 2 * m.ne), dtype=torch.complex128, device="cuda")
    print(f"rcs {name} right-hand sides {nrhs} directions {nd}", flush=True)
    out = cbfm.solve(mesh, med, h, Zr, inc, tol=1e-6, use_cmp=False, j_out=jt, dirs=dirs)
    j = jt.cpu().numpy()
    if nd:
        ref = excitation.rcs(m, j.T, dirs, w.k0, w.eta0)
    else:
        ref = excitation.monostatic_rcs(m, j.T, inc, w.k0, w.eta0)
    # both sum 21 terms a triangle in double; phases good to rounding times
    # k0 times the radius: 1e-12 of the largest value leaves a factor of 100
    assert np.abs(out["rcs"].reshape(ref.shape) - ref).max() < 1e-12 * np.abs(ref).max()
