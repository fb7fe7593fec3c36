"""CPU: the workgroups of 2D launches whose caller sets the segments' height
(tests/launchcheck: the library over a stand-in for the HIP runtime)."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "launchcheck", "wcnst_gridcheck.cpp")


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    from paper_1810_07806_amd import build
    if not os.path.exists(build.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("gridcheck") / "gridcheck")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O1", "-std=c++17", "-rdynamic",
                    "-I", build.INCLUDE, "-o", exe, SRC, "-ldl"], check=True, capture_output=True)

    def run(nx, ny, rows):
        r = subprocess.run([exe, build.LIB_PATH, str(nx), str(ny), str(rows)], check=True, capture_output=True,
                           text=True, timeout=60)
        return [int(x) for x in r.stdout.split()]
    return run


def _ceil(a, b):
    return -(-a // b)


@pytest.mark.parametrize("rows", [1, 2, 3, 5, 6])
@pytest.mark.parametrize("nx,ny", [(2048, 2048), (1024, 1024), (5000, 700)])
def test_low_segments_of_full_grids_are_joined(groups, nx, ny, rows):
    """A workgroup has the rows to fill its wavefronts, in whole segments."""
    n, reported = groups(nx, ny, rows)
    strips = _ceil(nx, 61)
    assert reported == rows
    assert n <= strips * _ceil(ny, 8)
    assert n in [strips * _ceil(ny, k * rows) for k in range(1, 17)]


SMALL = [(nx, ny, rows) for nx, ny in ((61, 61), (64, 128)) for rows in (1, 2, 3, 4, 5, 6, 7, 8, 13, 35, 64, 1000)]
LARGE = [(2048, 2048, rows) for rows in (4, 7, 8, 13, 35, 64, 1000)]


@pytest.mark.parametrize("nx,ny,rows", SMALL + LARGE)
def test_other_segments_are_as_set(groups, nx, ny, rows):
    """On grids that do not fill the CUs, and of every other height."""
    assert groups(nx, ny, rows) == [_ceil(nx, 61) * _ceil(ny, rows), rows]
