"""GPU: the stages that a profiled solve of a 1D line counts."""
from __future__ import annotations

import math

import pytest

from paper_1810_07806_amd import workloads as W

pytestmark = pytest.mark.gpu


# one launch; two (2048 steps each at most); a run of no final time in one and
# in two; a line of a launch per step; a failure
@pytest.mark.parametrize("nx,t_final,max_steps", [(200, 2.0, 10**6), (1000, 2.5, 10**6), (200, math.inf, 7),
                                                  (200, math.inf, 2049), (1000, math.inf, 7), (1000, 1.0, 1)])
def test_stages_of_a_short_line(nx, t_final, max_steps):
    from paper_1810_07806_amd.wcnst import E_MAX_STEPS, Solver, WcnstError
    d, U = W.advection_sine_square(nx)
    s = Solver(d)
    Ug = s.new_state(U)
    s.profile_enable(True)
    for _ in range(2):  # (a read starts over)
        s.reset()
        try:
            _, n = s.solve(Ug, t_final=t_final, max_steps=max_steps)
        except WcnstError as e:
            assert e.status == E_MAX_STEPS
            n = max_steps
        ms, stages = s.profile_read()
        assert n > 0 and stages == 3 * n and ms > 0.0
    s.step(Ug)
    assert s.profile_read()[1] == 3
    s.close()


def test_stages_up_to_a_failure():
    from paper_1810_07806_amd.wcnst import Solver, WcnstError
    d, U = W.riemann_1d(200, (1.0, -1.8, 0.4), (1.0, 1.8, 0.4))
    s = Solver(d)
    Ug = s.new_state(U)
    s.profile_enable(True)
    with pytest.raises(WcnstError):
        s.solve(Ug, t_final=1.0)
    n = s.status()["steps"]
    assert 0 < n < 10 and s.profile_read()[1] == 3 * n
    s.close()
