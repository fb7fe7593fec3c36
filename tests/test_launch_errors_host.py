"""CPU: every kernel launch of an entry point that fails is reported
(tests/launchcheck: the library over a stand-in for the HIP runtime)."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "launchcheck", "wcnst_launchcheck.cpp")
E_HIP = 4


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    from paper_1810_07806_amd import build
    if not os.path.exists(build.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("launchcheck") / "launchcheck")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O1", "-std=c++17", "-rdynamic",
                    "-I", build.INCLUDE, "-o", exe, SRC, "-ldl"], check=True, capture_output=True)

    def run(entry, ndim, nx):
        r = subprocess.run([exe, build.LIB_PATH, entry, str(ndim), str(nx)], check=True, capture_output=True,
                           text=True, timeout=60)
        return [int(x) for x in r.stdout.split()]
    return run


@pytest.mark.parametrize("ndim,nx", [(1, 200), (1, 700), (2, 40), (2, 200)])
@pytest.mark.parametrize("entry", ["step", "step_dt", "rhs", "solve", "noalloc"])
def test_a_failed_launch_is_reported(check, entry, ndim, nx):
    st = check(entry, ndim, nx)
    assert len(st) > 1 and st[-1] == 0
    assert st[:-1] == [E_HIP] * (len(st) - 1)
