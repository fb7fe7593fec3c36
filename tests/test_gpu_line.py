"""GPU: the 1D step kernels (a whole step per launch over tiles, many steps
of a short line in one workgroup) against the oracle, bit for bit, at the
sizes where their tiles and the choice between them change."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1810_07806_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 7


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    from paper_1810_07806_amd import wcnst
    wcnst.lib()
    return T


def _euler(nx, diff, bc):
    d, U = W.random_tube(np.random.default_rng(nx), nx)
    d.update(diff=diff, bc_x=bc)
    if bc == "fixed":
        d["fixed_x"] = (tuple(U[:, 0, 0]), tuple(U[:, 0, -1]))
    return d, U


def _burgers(nx, diff, bc):
    d = W.describe(ndim=1, system="burgers", nx=nx, x1=2.0, bc_x=bc, diff=diff)
    return d, (0.5 + np.sin(np.pi * W.coords(d))).reshape(1, 1, nx)


# smallest lines; one workgroup holding the line up to its last position, one
# past it; tiles of two threads a midpoint around their edges and up to the
# most (27904 cells, 256 tiles), one thread a midpoint past them
EULER = [(n, "mnd", bc) for n in (5, 57, 247, 248, 249, 474, 475) for bc in ("zero_gradient", "periodic", "reflect", "fixed")]
EULER += [(n, diff, "periodic") for n in (5, 61, 246, 247, 250, 251, 463) for diff in ("md", "hwcns")]
EULER += [(n, "mnd", bc) for n in (327, 328, 436, 27904, 27905) for bc in ("zero_gradient", "periodic", "reflect")]
SCALAR = [(n, diff, bc) for n in (5, 641, 1023, 1525, 1529, 1600) for diff, bc in
          (("mnd", "periodic"), ("md", "periodic"), ("hwcns", "zero_gradient"))]


@pytest.mark.parametrize("system,nx,diff,bc", [("euler", *c) for c in EULER] + [("burgers", *c) for c in SCALAR])
def test_steps_equal_the_oracle(orc, torch, system, nx, diff, bc):
    from paper_1810_07806_amd.wcnst import Solver
    d, U = (_euler if system == "euler" else _burgers)(nx, diff, bc)
    r = orc.solve(orc.problem(d), U, cfl=0.5, max_steps=STEPS)
    assert r["status"] == 0
    s = Solver(d)
    # in one call, and continued over three calls (odd and even step counts)
    for calls in ((STEPS,), (1, 4, STEPS - 5)):
        s.reset()
        Ug = s.new_state(U)
        for n in calls:
            s.solve(Ug, cfl=0.5, max_steps=n)
        st = s.status()
        assert st["steps"] == STEPS and st["t"] == r["t"]
        assert np.array_equal(Ug.cpu().numpy(), r["U"])
    # step by step
    s.reset()
    Ug = s.new_state(U)
    for _ in range(STEPS):
        s.step(Ug, cfl=0.5)
    assert s.status()["t"] == r["t"] and np.array_equal(Ug.cpu().numpy(), r["U"])
    s.close()


@pytest.mark.parametrize("u", [1.8, 2.5])
@pytest.mark.parametrize("nx", [200, 700])
def test_failure_is_the_oracles(orc, torch, nx, u):
    """A tube that loses positivity: stage, cell, time and steps."""
    from paper_1810_07806_amd.wcnst import Solver, WcnstError
    d, U = W.riemann_1d(nx, (1.0, -u, 0.4), (1.0, u, 0.4))
    r = orc.solve(orc.problem(d), U, cfl=0.5, t_final=0.1, max_steps=10000)
    assert r["status"] != 0
    s = Solver(d)
    Ug = s.new_state(U)
    with pytest.raises(WcnstError):
        s.solve(Ug, t_final=0.1)
    st = s.status()
    assert st["status"] != 0 and (st["bad_stage"], st["bad_cell"]) == (r["bad_stage"], r["bad_cell"])
    with pytest.raises(WcnstError):
        s.solve(Ug, t_final=0.2)
    s.close()


@pytest.mark.parametrize("nx", [100, 600])
def test_timed_solves_continue(orc, torch, nx):
    """To t = 0.02, then on to 0.05, equals the oracle's two solves."""
    from paper_1810_07806_amd.wcnst import Solver
    d, U = W.sod(nx)
    a = orc.solve(orc.problem(d), U, cfl=0.5, t_final=0.02, max_steps=10000)
    s = Solver(d)
    Ug = s.new_state(U)
    t, n = s.solve(Ug, t_final=0.02)
    assert t == a["t"] and n == a["steps"] and np.array_equal(Ug.cpu().numpy(), a["U"])
    t2, n2 = s.solve(Ug, t_final=0.05)
    assert abs(t2 - 0.05) <= 1e-13 and n2 > 0 and s.status()["steps"] == n + n2
    s.close()


@pytest.mark.parametrize("kw", [{}, dict(flux="lf", scheme="js"), dict(flux="vanleer", charwise=0)])
def test_batch_whose_tiles_change_equals_single_solves(torch, kw):
    """40 tubes of 1000 cells start with a thread a midpoint (400 pair tiles
    would not fit the CUs) and end, as most of them finish, with two."""
    from paper_1810_07806_amd.wcnst import Batch, Solver
    items = [W.random_tube(np.random.default_rng(i), 1000) for i in range(40)]
    for d, _ in items:
        d.update(kw)
    ts = [0.01 if i % 4 else 0.03 for i in range(40)]
    b = Batch([d for d, _ in items])
    b.set_tuning(4)
    U = b.pack([U for _, U in items])
    r = b.solve(U, ts)
    got = b.unpack(U)
    for i in (0, 1, 20, 39):
        s = Solver(items[i][0])
        V = s.new_state(items[i][1])
        t, n = s.solve(V, t_final=ts[i])
        assert r["status"][i] == 0 and r["steps"][i] == n and r["t"][i] == t
        assert np.array_equal(got[i], V.cpu().numpy().reshape(got[i].shape))
        s.close()
    b.close()
