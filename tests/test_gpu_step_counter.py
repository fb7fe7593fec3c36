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
@pytest.mark.parametrize("start", [-1, -2, -3, -100, 10**6, 2**28 // 3 - 2, 10**8, 2**40])
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


# a failure beyond the 2^28 stages that its record counts, and below zero:
# where it happened, and the state it leaves
@pytest.mark.parametrize("start", [-2, 10**8, 2**40])
@pytest.mark.parametrize("u,stage", [(1.8, 1), (2.5, 1)])
@pytest.mark.parametrize("nx", [200, 700])
def test_a_failure_at_any_step_number(orc, torch, nx, u, stage, start):
    from paper_1810_07806_amd.wcnst import Solver, WcnstError
    d, U = W.riemann_1d(nx, (1.0, -u, 0.4), (1.0, u, 0.4))
    p = orc.problem(d)
    r = orc.solve(p, U, cfl=0.5, max_steps=10)
    assert r["status"] != 0 and r["bad_stage"] % 3 == stage
    good = orc.solve(p, U, cfl=0.5, max_steps=r["bad_stage"] // 3)["U"]
    s = Solver(d)
    s.reset(0.0, start)
    Ug = s.new_state(U)
    with pytest.raises(WcnstError):
        s.solve(Ug, max_steps=10)
    st = s.status()
    assert st["status"] != 0 and st["bad_cell"] == r["bad_cell"]
    assert st["bad_stage"] == (3 * start + r["bad_stage"]) % 2**28
    assert np.array_equal(Ug.cpu().numpy(), good)
    s.close()
