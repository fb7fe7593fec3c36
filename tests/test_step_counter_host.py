"""CPU check of what the device code does with the step counter, which a
caller may start from any value (wcnst_reset)."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "linecheck", "wcnst_stepcheck.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1810_07806_amd", "csrc")
STARTS = [0, 1, 7, -1, -2, -3, -100, 2**28 // 3 - 2, 10**8, 2**40, -(2**40)]


@pytest.fixture(scope="module")
def sc(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("stepcheck") / "libstepcheck.so")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", CSRC, "-o", lib, SRC], check=True, capture_output=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("start", STARTS)
def test_speed_slots_stay_in_their_array(sc, start):
    """Three in turn, whatever the counter's sign."""
    sc.sc_speed_slot.argtypes = [ctypes.c_longlong]
    slots = [sc.sc_speed_slot(n) for n in range(start, start + 9)]
    assert set(slots) == {0, 1, 2}
    assert all(b == (a + 1) % 3 for a, b in zip(slots, slots[1:]))


@pytest.mark.parametrize("start", STARTS)
def test_a_failure_names_its_own_step(sc, start):
    sc.sc_bad_stage.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong]
    sc.sc_bad_stage.restype = ctypes.c_uint
    for stage in range(3):
        for cell in (0, 2**34 - 1):
            assert sc.sc_bad_stage(start, stage, cell, start) == stage
            for other in (-5, -1, 1, 2, 1000):
                assert sc.sc_bad_stage(start, stage, cell, start + other) > 2
