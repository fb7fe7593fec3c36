"""GPU: calls on a 1D solver whose last step failed (the status is sticky
until a reset) leave the caller's state alone."""
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


def _failing_step(orc, nx, before, stage):
    """A tube, and a CFL number at which the step after `before` small ones
    fails in the given stage."""
    for d, U in (W.sod(nx), W.lax(nx), W.riemann_1d(nx, (1.0, 5.0, 0.1), (1.0, -5.0, 0.1))):
        p = orc.problem(d)
        V = U
        for _ in range(before):
            V, bad, _, _ = orc.rk3_step(p, V, 0.1 / orc.max_speed(p, V))
            assert bad == 0
        for cfl in np.arange(0.5, 3.0, 0.05):
            _, bad, bad_stage, _ = orc.rk3_step(p, V, float(cfl) / orc.max_speed(p, V))
            if bad != 0 and bad_stage == stage:
                return d, U, V, float(cfl)
    raise AssertionError("no such step")


# a line in one workgroup, one of several tiles; the failing step at either
# parity, in a step call and in a run
@pytest.mark.parametrize("stage", [0, 1, 2])
@pytest.mark.parametrize("before", [1, 2])
@pytest.mark.parametrize("nx", [200, 700])
@pytest.mark.parametrize("how", ["step", "solve"])
def test_calls_after_a_failure_leave_the_state(orc, torch, nx, before, stage, how):
    from paper_1810_07806_amd.wcnst import Solver, WcnstError
    d, U0, start, cfl = _failing_step(orc, nx, before, stage)
    s = Solver(d)
    U = s.new_state(U0)
    if how == "step":
        for _ in range(before):
            s.step(U, cfl=0.1)
        s.step(U, cfl=cfl)
    else:
        s.solve(U, cfl=0.1, max_steps=before)
        with pytest.raises(WcnstError):
            s.solve(U, cfl=cfl, max_steps=3)
    st = s.status()
    assert st["status"] != 0 and st["bad_stage"] == 3 * before + stage
    left = U.cpu().numpy()
    if stage < 2:  # (a failure in the last stage leaves its output)
        assert np.array_equal(left, start)
    fresh = s.new_state(U0)
    for V, want in ((U, left), (fresh, U0)):
        for _ in range(3):
            s.step(V, cfl=0.1)
            assert np.array_equal(V.cpu().numpy(), want, equal_nan=True)
        for kw in (dict(max_steps=0), dict(max_steps=2), dict(t_final=1.0), dict(max_steps=0)):
            with pytest.raises(WcnstError):
                s.solve(V, cfl=0.1, **kw)
            assert np.array_equal(V.cpu().numpy(), want, equal_nan=True)
            s.step(V, cfl=0.1)
            assert np.array_equal(V.cpu().numpy(), want, equal_nan=True)
    # a reset clears the status and the line runs on
    s.reset()
    s.solve(fresh, cfl=0.1, max_steps=before)
    assert np.array_equal(fresh.cpu().numpy(), start) and s.status()["status"] == 0
    s.close()


@pytest.mark.parametrize("nx", [200, 700])
def test_a_call_of_no_steps_leaves_the_state(torch, nx):
    from paper_1810_07806_amd.wcnst import Solver
    d, U0 = W.sod(nx)
    s = Solver(d)
    U = s.new_state(U0)
    for n in (0, 1, 0, 2, 0):
        before = U.cpu().numpy()
        _, took = s.solve(U, max_steps=n)
        assert took == n and np.array_equal(U.cpu().numpy(), before) == (n == 0)
    s.close()
