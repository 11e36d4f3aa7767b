"""CBFs kept below the rounding level of the core (delta_svd = 0): with every
third generating wave a combination of the two before it, a third of the kept
functions stand for no direction.  Their right vectors must still be
orthogonal to the others', so that their coefficients C^J = J^J V vanish up to
the dependence's own rounding, and the others are those of a build that
truncates (Sec. III-B)."""
import numpy as np
import pytest

from conftest import oracle_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells, directions, max_L", [(1, 8, 0), (8, 8, 0), (8, 7, 19), (8, 25, 0), (1, 40, 0), (1, 40, 100)])
def test_dependent_waves(cells, directions, max_L):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from oracle import cbf as ocbf
    from paper_2111_11058_amd import cbfm
    from synth import configs
    P = oracle_problem("c1")
    w, m = P["w"], P["m"]
    gen = []
    for row in configs.random_incidences(directions, 3):
        k, p = row[:3], row[3:]
        q = np.cross(k, p)
        gen += [np.concatenate([k, t]) for t in (p, q, 0.6 * p + 0.8 * q)]
    gen = np.array(gen)
    rank = 2 * directions
    eb = np.asarray(w.edge_block if cells == 8 else np.zeros(m.ne), np.int32)
    mesh = cbfm.Mesh(w.V, w.T, eb, cells)
    med = cbfm.Medium.make(w.k0, w.eta0, w.eps_r, w.mu_r)
    print(f"dependent waves cells {cells} directions {directions} max_L {max_L}", flush=True)
    full = cbfm.build_cbf(mesh, med, gen, 0.0, max_L=max_L)
    some = cbfm.build_cbf(mesh, med, gen, 1e-6)
    CM, CJ = full.export()
    G = ocbf.rwg_gram(m)
    o = o1 = 0
    for b in range(cells):
        s, t = full.sigma[o:o + full.L[b]], some.sigma[o1:o1 + some.L[b]]
        o, o1 = o + full.L[b], o1 + some.L[b]
        # every function asked for, less exact zeros (none is a third of the waves at most)
        assert full.L[b] >= min(rank, max_L or rank)
        k = min(len(s), len(t))
        assert np.abs(s[:k] - t[:k]).max() < 1e-12 * s[0]
        # the third waves depend on the others to the rounding of the solves,
        # 1e-16 times the condition number of Z_mm, some 1e6
        assert s[rank:].max(initial=0.0) < 1e-12 * s[0]
        size = np.linalg.norm(CJ[b], axis=0)
        print(b, len(s), len(t), size[rank:].max(initial=0.0) / size.max())
        assert size[rank:].max(initial=0.0) < 1e-9 * size.max()
        ix = np.flatnonzero(eb == b)
        D = CM[b][:, :k].conj().T @ G[np.ix_(ix, ix)] @ CJ[b][:, :k]
        assert np.abs(D - np.diag(s[:k])).max() < 1e-8 * s[0]
