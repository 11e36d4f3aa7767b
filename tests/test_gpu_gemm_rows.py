"""The vector-unit product of few columns at its edges, called as the library
calls it (cbfm::zgemm_batched with one descriptor): odd and even numbers of
rows, contraction lengths around its 256 threads and their pairs, 2 to 8
columns, every pair of operations that it takes, complex factors, added
results, both layouts of the result, padded leading dimensions; against numpy,
nothing written beside the result."""
import ctypes as C
import os
import re

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc", "gemm.hip")
OP_N, OP_T, OP_C, OP_R = range(4)
ZGEMM = "_ZN4cbfm13zgemm_batchedERSt6vectorINS_8GemmDescESaIS1_EEP12ihipStream_tPS0_IS3_SaIS3_EE"


class Desc(C.Structure):
    _fields_ = [("A", C.c_void_p), ("B", C.c_void_p), ("C", C.c_void_p), ("lda", C.c_int64), ("ldb", C.c_int64),
                ("ldc", C.c_int64), ("M", C.c_int64), ("N", C.c_int64), ("K", C.c_int64), ("opA", C.c_int32),
                ("opB", C.c_int32), ("alpha_re", C.c_double), ("alpha_im", C.c_double), ("accumulate", C.c_int32),
                ("transC", C.c_int32), ("tile_start", C.c_int64)]


class Vector(C.Structure):  # std::vector<GemmDesc>
    _fields_ = [("begin", C.c_void_p), ("end", C.c_void_p), ("cap", C.c_void_p)]


def _product(M, N, K, opA, opB, alpha, acc, trans, seed):
    from paper_2111_11058_amd import cbfm
    rng = np.random.default_rng(seed)
    z = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    pad = 3
    A, B = z(M, K + pad), z(N, K + pad)
    C0 = z(*((N, M + pad) if trans else (M, N + pad)))
    dev = [torch.tensor(x, device="cuda") for x in (A, B, C0)]
    d = (Desc * 1)(Desc(dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), K + pad, K + pad, C0.shape[1], M, N, K, opA, opB,
                        alpha.real, alpha.imag, acc, trans, 0))
    at = C.addressof(d)
    v = Vector(at, at + C.sizeof(Desc), at + C.sizeof(Desc))
    torch.cuda.synchronize()
    f = getattr(cbfm.lib(), ZGEMM)
    f.restype = None
    f(C.byref(v), C.c_void_p(None), C.c_void_p(None))
    torch.cuda.synchronize()
    a = A[:, :K].conj() if opA == OP_R else A[:, :K]
    b = B[:, :K].conj() if opB == OP_C else B[:, :K]
    P = alpha * (a @ b.T)
    want = C0.copy()
    part = want[:N, :M] if trans else want[:M, :N]
    P = P.T if trans else P
    part[...] = part + P if acc else P
    got = dev[2].cpu().numpy()
    edge = np.ones(C0.shape, bool)
    edge[:, :C0.shape[1] - pad] = False
    assert np.array_equal(got[edge], C0[edge])
    # a sum of K products in any order, and the factor: (K + 8) roundings of the sizes
    size = (np.abs(a) @ np.abs(b).T) * abs(alpha)
    size = size.T if trans else size
    err = np.abs(got - want)[~edge].reshape(part.shape)
    assert np.all(err <= (2 * K + 16) * 2.0 ** -52 * (size + np.abs(part)))
    return got


def test_shape_number():
    names = re.findall(r"\bGV_\w+", re.search(r"enum \{(\s+GV_TILE4 = 0.*?)\};", open(SRC).read(), re.S).group(1))
    assert names[11] == "GV_ROWS" and names[12] == "GV_COUNT"


@pytest.mark.parametrize("opA, opB", [(OP_N, OP_T), (OP_N, OP_C), (OP_R, OP_T), (OP_R, OP_C)])
@pytest.mark.parametrize("M, K", [(1, 1), (2, 255), (7, 256), (33, 257), (5, 511), (12, 512), (3, 513), (129, 1030), (640, 640)])
def test_edges(M, K, opA, opB, monkeypatch):
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    print("few columns", M, K, opA, opB, flush=True)
    own = other = 0
    for N in range(2, 10):  # (9: another shape takes it)
        for acc, trans, alpha in ((0, 1, 1.0 + 0j), (0, 0, -1.0 + 0j), (1, 0, 0.75 - 0.5j), (1, 1, 2.0 + 1j)):
            monkeypatch.setenv("CBFM_GEMM_SHAPE", "11")
            x = _product(M, N, K, opA, opB, alpha, acc, trans, 100 * N + M)
            monkeypatch.setenv("CBFM_GEMM_SHAPE", "1")
            y = _product(M, N, K, opA, opB, alpha, acc, trans, 100 * N + M)
            if N < 9:
                own += not np.array_equal(x, y)
            else:
                other += not np.array_equal(x, y)
    # the sums' orders differ where there is more than a handful of terms, so
    # that equal bits everywhere would mean that another kernel ran
    assert own > 0 or K < 16
    assert other == 0
