"""CPU check that every position a stage of a 1D tile forms has a thread
(tests/linecheck)."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "linecheck", "wcnst_tilethreads.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1810_07806_amd", "csrc")


@pytest.fixture(scope="module")
def tt(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("tilethreads") / "libtilethreads.so")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", CSRC, "-o", lib, SRC], check=True, capture_output=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("diff,pair", [(0, 0), (0, 1), (1, 0), (2, 0)])
@pytest.mark.parametrize("bc", [0, 1, 2, 3])
def test_every_formed_position_has_a_thread(tt, bc, diff, pair):
    threads = tt.tt_threads()
    for nx in list(range(5, 60000)) + [100003, 1000001]:
        assert tt.tt_most(nx, bc, diff, pair) <= threads, nx


@pytest.mark.parametrize("bc", [0, 1, 2, 3])
def test_lines_of_one_and_two_wavefronts_fit_them(tt, bc):
    """Up to 56 and 120 cells: every position and midpoint has a thread, and
    every position its place."""
    for nx in range(5, 121):
        room = 64 if nx <= 56 else 128
        assert 0 < tt.tt_whole(nx, bc) <= room and tt.tt_most(nx, bc, 0, 0) <= room, nx
