"""Host rules of the library that are plain C++, compiled and called on the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from helpers import ROOT


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "rules.cpp"
    src.write_text('#include "stencil.h"\n'
                   'extern "C" int within(const int32_t *nc, int64_t n, int64_t most) {\n'
                   '  return ljmd::mean_stencil_within(nc, n, most);\n}\n')
    lib = d / "rules.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2109_09056_amd", "csrc"), "-o", str(lib), str(src)],
                   check=True)
    f = ctypes.CDLL(str(lib)).within
    f.argtypes = [ctypes.POINTER(ctypes.c_int32), ctypes.c_int64, ctypes.c_int64]
    return lambda nc, n, most: bool(f((ctypes.c_int32 * 3)(*nc), n, most))


@pytest.mark.parametrize("nc", [(1, 1, 1), (2, 2, 2), (1, 2, 9), (2, 3, 3), (3, 3, 3), (4, 5, 7)])
def test_mean_stencil_counts_distinct_cells(rules, nc):
    """Against the stencils written out: distinct cells (mod nc) around each cell, the mean of
    their atoms for n atoms spread evenly; 256 atoms in 2 x 2 x 2 cells have 256 candidates."""
    per_cell = [{tuple((c[k] + o[k]) % nc[k] for k in range(3))
                 for o in np.ndindex(3, 3, 3)} for c in np.ndindex(*nc)]
    mean_cells = np.mean([len(s) for s in per_cell])
    cells = int(np.prod(nc))
    for n in (1, 256, 864, 100000):
        mean = n / cells * mean_cells
        for most in (int(np.floor(mean)) - 1, int(np.ceil(mean)), int(np.ceil(mean)) + 1):
            assert rules(nc, n, most) == (mean <= most), (n, most)
