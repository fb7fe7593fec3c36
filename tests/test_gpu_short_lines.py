"""GPU: launches over thousands of short lines, which take workgroups of one
or two wavefronts, against the oracle bit for bit."""
from __future__ import annotations

import math

import numpy as np
import pytest

from paper_1810_07806_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 5


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    from paper_1810_07806_amd import wcnst
    wcnst.lib()
    return T


def _lines(sizes, kw):
    """A line of each size with each kind of ends."""
    out = []
    for nx in sizes:
        for bc in ("zero_gradient", "periodic", "reflect", "fixed"):
            d, U = W.random_tube(np.random.default_rng(nx), nx)
            d.update(kw, bc_x=bc)
            if bc == "fixed":
                d["fixed_x"] = (tuple(U[:, 0, 0]), tuple(U[:, 0, -1]))
            out.append((d, U))
    return out


# one wavefront up to its last position, two, and the full tile past them; the
# fewest lines that take them, and the most that do not
@pytest.mark.parametrize("count,sizes", [(1025, (5, 8, 33, 56)), (1025, (6, 57, 64)), (1100, (56, 119, 120)),
                                         (1100, (20, 120, 121)), (1024, (5, 56))])
@pytest.mark.parametrize("kw", [{}, dict(flux="lf", scheme="js", charwise=0), dict(flux="vanleer", q=4)])
def test_short_lines_equal_the_oracle(orc, torch, count, sizes, kw):
    from paper_1810_07806_amd.wcnst import Batch, Pool
    kinds = _lines(sizes, kw)
    want = [orc.solve(orc.problem(d), U, cfl=0.3, max_steps=STEPS) for d, U in kinds]
    assert all(r["status"] == 0 for r in want)
    pick = [kinds[i % len(kinds)] for i in range(count)]
    b = Batch([d for d, _ in pick])
    b.set_tuning(2)
    U = b.pack([U for _, U in pick])
    r = b.solve(U, math.inf, cfl=0.3, max_steps=STEPS)
    got = b.unpack(U)
    for i in range(count):
        w = want[i % len(kinds)]
        assert (r["status"][i], r["steps"][i], r["t"][i]) == (0, STEPS, w["t"])
        assert np.array_equal(got[i], w["U"].reshape(got[i].shape))
    b.close()
    # the same lines as requests of a pool
    p = Pool(scheme=dict(kw), capacity=count)
    bufs, slots = [], []
    for d, U0 in pick:
        V = torch.zeros((3, U0.size), dtype=torch.float64, device="cuda")
        V[0] = torch.as_tensor(U0.reshape(-1))
        bufs.append(V)
        slots.append(p.admit(d, V[0], V[1], V[2], 1e3, cfl=0.3))
    for n in (2, STEPS - 2):
        assert p.tick(n) == count
    for i, (V, slot) in enumerate(zip(bufs, slots)):
        w, res = want[i % len(kinds)], p.result(slot)
        assert (res["status"], res["steps"], res["t"]) == (0, STEPS, w["t"])
        assert np.array_equal(V[0].cpu().numpy(), w["U"].reshape(-1))
    p.close()


@pytest.mark.parametrize("nx", [50, 100])
def test_a_failure_among_short_lines_stays_its_own(orc, torch, nx):
    from paper_1810_07806_amd.wcnst import Batch
    good = W.sod(nx)
    bad = W.riemann_1d(nx, (1.0, -2.5, 0.4), (1.0, 2.5, 0.4))
    items = [bad if i == 700 else good for i in range(1100)]
    rg = orc.solve(orc.problem(good[0]), good[1], cfl=0.5, t_final=0.05)
    rb = orc.solve(orc.problem(bad[0]), bad[1], cfl=0.5, t_final=0.05)
    assert rg["status"] == 0 and rb["status"] != 0
    b = Batch([d for d, _ in items])
    U = b.pack([u for _, u in items])
    r = b.solve(U, 0.05)
    stage, cell = b.bad_cells()
    for i in range(1100):
        if i == 700:
            assert r["status"][i] != 0 and (stage[i], cell[i]) == (rb["bad_stage"], rb["bad_cell"])
        else:
            assert (r["status"][i], r["steps"][i], r["t"][i]) == (0, rg["steps"], rg["t"])
    got = b.unpack(U)
    assert np.array_equal(got[0], rg["U"].reshape(got[0].shape))
    assert np.array_equal(got[1099], got[0])
    b.close()
