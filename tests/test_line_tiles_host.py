"""CPU check of the 1D step kernels' index geometry (tests/linecheck): every
tile of lines from the smallest to past several tiles, each boundary kind and
difference."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "linecheck", "wcnst_linecheck.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1810_07806_amd", "csrc")


@pytest.fixture(scope="module")
def lc(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("linecheck") / "liblinecheck.so")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", CSRC, "-o", lib, SRC], check=True, capture_output=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("diff,pair", [(0, 0), (0, 1), (1, 0), (2, 0)])
@pytest.mark.parametrize("bc", [0, 1, 2, 3])
def test_line_tiles_stay_in_their_positions(lc, bc, diff, pair):
    sizes = list(range(5, 1100)) + [2047, 2048, 4096, 16383, 16384, 54321, 56169, 100003, 1000001]
    for nx in sizes:
        assert lc.lc_check(nx, bc, diff, pair) == 0, nx
