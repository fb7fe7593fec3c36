"""GPU: the 2D stage (short segments whole, longer ones four rows at a time)
against the oracle, bit for bit, at the edges of its strips, segments and
turns."""
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


# whole segments of one row up to the most (12: two staged rows per wavefront
# from 5, two midpoint rows from 5, three from 11), one row past it, and whole
# turns of a longer segment
@pytest.mark.parametrize("rows", [1, 3, 4, 5, 8, 9, 11, 12, 13, 16, 0])
@pytest.mark.parametrize("nx,ny", [(5, 5), (61, 8), (62, 9), (123, 14)])
@pytest.mark.parametrize("bc", ["zero_gradient", "periodic", "reflect"])
def test_rhs_flags_and_steps_equal_the_oracle(orc, torch, nx, ny, rows, bc):
    from paper_1810_07806_amd.wcnst import Solver, split_flags
    d, U = W.random_euler2d(np.random.default_rng(nx), nx, ny)
    d.update(bc_x=bc, bc_y=bc)
    if bc == "reflect":
        d["gravity"] = 0.5
    p = orc.problem(d)
    Ro, fo, _ = orc.rhs(p, U, flags=True)
    s = Solver(d)
    s.set_tuning(rows)
    Ug = s.new_state(U)
    R, fl = s.rhs(Ug, flags=True)
    assert np.array_equal(R.cpu().numpy(), Ro)
    for a, b in zip(split_flags(d, fl.cpu().numpy()), fo):
        # (equal outside ties at the cut-off, which these states do not have)
        assert np.array_equal(a, b)
    r = orc.solve(p, U, cfl=0.5, max_steps=3)
    s.solve(Ug, cfl=0.5, max_steps=3)
    assert s.status()["t"] == r["t"] and np.array_equal(Ug.cpu().numpy(), r["U"])
    s.close()


# more workgroups than the device takes at once: short segments by turns (4),
# whole turns (16) and a last turn of one row (13)
@pytest.mark.parametrize("rows", [4, 13, 16])
def test_crowded_launches_equal_the_oracle(orc, torch, rows):
    from paper_1810_07806_amd.wcnst import Solver
    d, U = W.random_euler2d(np.random.default_rng(7), 400, 301)
    d.update(bc_x="periodic", bc_y="zero_gradient")
    p = orc.problem(d)
    r = orc.solve(p, U, cfl=0.5, max_steps=2)
    s = Solver(d)
    s.set_tuning(rows)
    Ug = s.new_state(U)
    s.solve(Ug, cfl=0.5, max_steps=2)
    assert s.status()["t"] == r["t"] and np.array_equal(Ug.cpu().numpy(), r["U"])
    s.close()
