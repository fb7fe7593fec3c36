"""GPU: a timed 2D solve goes on from where the one before it ended, whether
an even or an odd number of steps were queued past its final time."""
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


# 1 to 9 steps in the first solve: its last look-ahead chunk has every parity
@pytest.mark.parametrize("t1", [0.003, 0.005, 0.008, 0.011, 0.014, 0.017, 0.02, 0.03])
def test_timed_2d_solves_continue(orc, torch, t1):
    from paper_1810_07806_amd.wcnst import Solver
    d, U = W.riemann2d_config3(40)
    p = orc.problem(d)
    a = orc.solve(p, U, cfl=0.5, t_final=t1)
    b = orc.solve(p, a["U"], cfl=0.5, t0=a["t"], t_final=0.05)
    c, bad, _, _ = orc.rk3_step(p, b["U"], 0.5 / orc.max_speed(p, b["U"]))
    assert a["status"] == b["status"] == bad == 0
    s = Solver(d)
    Ug = s.new_state(U)
    assert s.solve(Ug, t_final=t1) == (a["t"], a["steps"])
    assert np.array_equal(Ug.cpu().numpy(), a["U"])
    assert s.solve(Ug, t_final=0.05) == (b["t"], b["steps"])
    assert np.array_equal(Ug.cpu().numpy(), b["U"])
    s.step(Ug)
    assert s.status()["steps"] == a["steps"] + b["steps"] + 1
    assert np.array_equal(Ug.cpu().numpy(), c)
    s.close()
