"""Solves of many short cycles, whose end by their length leaves a copy of the
convergence flags in flight: restarts of one chunk of iterations and of two in
the mixed, compressed-basis, s-step and plain forms.  Every solve goes on
until the true residual is at the tolerance, and repeats give the same counts."""
import numpy as np
import pytest

from test_gpu_krylov_forms import _MESH, _system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [4, 8])
@pytest.mark.parametrize("how", [dict(inner_fp32=True, inner_tol=1e-2), dict(basis_fp32=True, inner_tol=1e-2),
                                 dict(sstep=4), dict()], ids=["mixed", "basis", "sstep", "plain"])
def test_short_cycles(how, restart):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    from synth import configs
    h, n, Zr, _, _ = _system(2)
    Zt = torch.tensor(Zr, dtype=torch.complex128, device="cuda")
    inc = configs.random_incidences(5, 5)
    counts = []
    for _ in range(12):
        o = cbfm.solve(_MESH["mesh"], _MESH["med"], h, Zt, inc, tol=1e-10, max_iter=400, restart=restart, use_cmp=False, **how)
        assert o["status"] == "OK" and np.all(o["relres"] <= 1e-10), (o["status"], o["iters"], o["relres"])
        counts.append(o["iters"].tolist())
    print(how, restart, counts[0], flush=True)
    assert all(c == counts[0] for c in counts)


@pytest.mark.parametrize("how", [dict(), dict(inner_fp32=True), dict(basis_fp32=True)], ids=["plain", "mixed", "basis"])
@pytest.mark.parametrize("nrhs, restart", [(1, 4), (3, 7), (2, 13), (70, 40), (3, 256)])
def test_captured_chunks(nrhs, restart, how):
    """Captured chunks of four iterations (their column steps once a chunk),
    the rest of a cycle uncaptured: the counts of the uncaptured solve within
    one, and its residual."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    from synth import configs
    h, n, Zr, _, _ = _system(2)
    Zt = torch.tensor(Zr, dtype=torch.complex128, device="cuda")
    inc = configs.random_incidences(nrhs, 5)
    a, b = [cbfm.solve(_MESH["mesh"], _MESH["med"], h, Zt, inc, tol=1e-11, max_iter=400, restart=restart, use_cmp=False,
                       use_graph=g, **how) for g in (False, True)]
    print("captured", nrhs, restart, how, a["iters"].max(), b["iters"].max(), flush=True)
    assert a["status"] == "OK" and b["status"] == "OK" and np.all(b["relres"] <= 1e-11)
    assert np.abs(a["iters"] - b["iters"]).max() <= 1
