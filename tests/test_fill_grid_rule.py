"""The regular fill's choice of the grid's faster dimension, compiled from its
source for the host: where rows vary fastest, the columns' blocks lie along
the grid's second dimension, which holds 65,535; a mesh of any size is filled
(the rows of one launch are limited elsewhere)."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc", "fill.hip")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_columns_fit_the_grid(tmp_path):
    src = open(SRC).read()
    rule = re.search(r"static bool fill_rows_first\(.*?\n}\n", src, re.S).group(0)
    assert "too many column triangles" not in src
    cpp = tmp_path / "rule.cpp"
    cpp.write_text("#include <cstdint>\n" + rule + 'extern "C" int rows_first(long n, int fp64) { return fill_rows_first(n, fp64 != 0); }\n')
    so = str(tmp_path / "rule.so")
    subprocess.run(["g++", "-shared", "-fPIC", str(cpp), "-o", so], check=True)
    f = ctypes.CDLL(so).rows_first
    f.argtypes = [ctypes.c_long, ctypes.c_int]
    sizes = [1, 255, 256, 512, 513, 1728, 19968, 65535 * 256 - 1, 65535 * 256, 65535 * 256 + 1, 2 ** 31 - 1]
    for fp64 in (0, 1):
        for n in sizes:
            assert not f(n, fp64) or (n + 255) // 256 <= 65535, n
    assert f(19968, 1) and f(65535 * 256, 1) and not f(65535 * 256 + 1, 1)
