"""GPU: a 1D solve is the same from whatever value its step counter starts."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1810_07806_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    from paper_1810_07806_amd import wcnst
    wcnst.lib()
    return T


# a line in one workgroup, one of several tiles
@pytest.mark.parametrize("start", [-1, -2, -3, -100, 10**6])
@pytest.mark.parametrize("nx", [200, 700])
def test_any_first_step_number(orc, torch, nx, start):
    from paper_1810_07806_amd.wcnst import Solver
    d, U = W.sod(nx)
    r = orc.solve(orc.problem(d), U, cfl=0.5, max_steps=7)
    s = Solver(d)
    s.reset(0.0, start)
    Ug = s.new_state(U)
    s.solve(Ug, max_steps=4)
    for _ in range(3):
        s.step(Ug)
    st = s.status()
    assert (st["status"], st["steps"], st["t"]) == (0, start + 7, r["t"])
    assert np.array_equal(Ug.cpu().numpy(), r["U"])
    s.close()
