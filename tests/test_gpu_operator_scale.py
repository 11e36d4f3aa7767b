"""The solvers do not depend on the operator's units: Z_r times a factor, far
from 1 but within float's range, takes the same iterations to the same
residual in every Krylov form (a body given in metres instead of wavelengths
scales Z_r by many orders of magnitude)."""
import numpy as np
import pytest

from test_gpu_krylov_forms import _MESH, _system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("how", [dict(inner_fp32=True), dict(inner_fp32=True, use_graph=True), dict(basis_fp32=True),
                                 dict(), dict(sstep=8), dict(block=3)],
                         ids=["mixed", "mixed-graph", "basis", "plain", "sstep", "block"])
def test_scaled_operator(how):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_11058_amd import cbfm
    from synth import configs
    h, n, Zr, _, _ = _system(2)
    inc = configs.random_incidences(3, 5)
    first = None
    for scale in (1.0, 2.0 ** -73, 2.0 ** 73, 2.0 ** -100, 2.0 ** 100):
        o = cbfm.solve(_MESH["mesh"], _MESH["med"], h, torch.tensor(Zr * scale, device="cuda"), inc, tol=1e-10, max_iter=300,
                       restart=n, use_cmp=False, **how)
        print(how, scale, o["status"], o["iters"], o["relres"].max(), flush=True)
        assert o["status"] == "OK" and np.all(o["relres"] <= 1e-10)
        first = o["iters"] if first is None else first
        assert np.abs(o["iters"] - first).max() <= 1
