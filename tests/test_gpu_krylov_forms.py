"""The Krylov forms' kernels by their sizes: s-step cycles with the block of
vectors in LDS or not (S n double complex values against a compute unit's
160 KB: n of about 1,100 for S = 8 and 2,470 for S = 4), block GMRES with
full, odd and single-column groups, and plain cycles whose lengths fall short
of, meet and pass the chunks of four iterations.  Random CBFs and Z_r = I + E (E seeded,
spectral norm about 0.4), so that any size has an exact answer by LU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

_MESH = {}


def _system(L):
    """Mesh, medium, CBFs (L per cell, 64 cells), Z_r and C^JM, C^MJ."""
    from oracle import mesh as om, reduced
    from oracle.cbf import CBFSet
    from paper_2111_11058_amd import cbfm
    from synth import configs
    if not _MESH:
        w = configs.sphere_c3()
        _MESH.update(w=w, m=om.build(w.V, w.T), mesh=cbfm.Mesh(w.V, w.T, w.edge_block, w.nblocks),
                     med=cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r))
    w, m = _MESH["w"], _MESH["m"]
    cells = [np.flatnonzero(np.asarray(w.edge_block) == a) for a in range(w.nblocks)]
    CM = [configs.random_complex((len(ix), L), 100 + a) for a, ix in enumerate(cells)]
    CJ = [configs.random_complex((len(ix), L), 900 + a) for a, ix in enumerate(cells)]
    sigma = [np.ones(L) for _ in cells]
    cb = CBFSet(cells=cells, CM=CM, CJ=CJ, sigma=sigma, sigma_all=sigma)
    h = cbfm.cbf_import(_MESH["mesh"], CM, CJ, sigma)
    n = h.n_cbf
    Zr = np.eye(n) + configs.random_complex((n, n), 27) * (0.4 / (2.0 * np.sqrt(n)))
    return h, n, Zr, *reduced.cbf_matrices(cb, m.ne)


def _check(h, Zr, CJM, CMJ, inc, restart=None, **how):
    import torch
    from oracle import excitation
    from paper_2111_11058_amd import cbfm
    w, m = _MESH["w"], _MESH["m"]
    jref = CMJ @ np.linalg.solve(Zr, CJM.conj().T @ excitation.rhs(m, inc, w.k0, w.eta0))
    jt = torch.zeros((len(inc), 2 * m.ne), dtype=torch.complex128, device="cuda")
    Zt = torch.tensor(Zr, dtype=torch.complex128, device="cuda")
    print("solve", how, "n", h.n_cbf, "right-hand sides", len(inc), flush=True)
    out = cbfm.solve(_MESH["mesh"], _MESH["med"], h, Zt, inc, tol=1e-12, max_iter=300,
                     restart=restart or h.n_cbf, use_cmp=False, j_out=jt, **how)
    e = np.linalg.norm(jt.cpu().numpy().T - jref) / np.linalg.norm(jref)
    print(out["iters"], out["relres"].max(), e)
    assert out["status"] == "OK" and np.all(out["relres"] <= 1e-12)
    assert e < 1e-9


@pytest.mark.parametrize("S, L, nrhs", [(8, 8, 3), (8, 9, 3), (4, 9, 1), (4, 19, 2), (4, 20, 2)])
def test_sstep_sizes(S, L, nrhs):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from synth import configs
    h, n, Zr, CJM, CMJ = _system(L)
    _check(h, Zr, CJM, CMJ, configs.random_incidences(nrhs, 5), sstep=S)


@pytest.mark.parametrize("block, nrhs", [(2, 3), (3, 3), (7, 15), (16, 16), (17, 17), (31, 31), (32, 33)])
def test_block_sizes(block, nrhs):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from synth import configs
    h, n, Zr, CJM, CMJ = _system(5)
    _check(h, Zr, CJM, CMJ, configs.random_incidences(nrhs, 5), block=block)


@pytest.mark.parametrize("L, nrhs, restart", [(1, 1, 1), (1, 2, 3), (1, 1, 4), (2, 5, 5), (1, 3, 8), (5, 65, 9),
                                              (5, 1, 640), (1, 130, 128), (9, 2, 13)])
def test_plain_cycles(L, nrhs, restart):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    from synth import configs
    h, n, Zr, CJM, CMJ = _system(L)
    inc = configs.random_incidences(nrhs, 5)
    _check(h, Zr, CJM, CMJ, inc, restart)
    # an iteration limit inside a chunk stops there, unconverged
    for lim in (1, 6):
        o = cbfm.solve(_MESH["mesh"], _MESH["med"], h, torch.tensor(Zr, device="cuda"), inc, tol=1e-30, max_iter=lim,
                       restart=restart, use_cmp=False)
        assert o["status"] == "E_NOCONV" and np.all(o["iters"] == lim) and np.all(o["relres"] < 1)


@pytest.mark.parametrize("L, nrhs", [(1, 2), (1, 3), (2, 4), (2, 5), (5, 7), (9, 8), (1, 9)])
def test_few_column_product(L, nrhs, monkeypatch):
    """The vector-unit product of 2 to 8 columns, forced (9: not taken)."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from synth import configs
    monkeypatch.setenv("CBFM_GEMM_SHAPE", "11")
    h, n, Zr, CJM, CMJ = _system(L)
    _check(h, Zr, CJM, CMJ, configs.random_incidences(nrhs, 5))
