"""GPU: low segments of a full grid, several to a workgroup, against the
oracle bit for bit: flags, right-hand side and steps, alone and in a pool."""
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


@pytest.mark.parametrize("rows", [1, 2, 3, 5, 6])
def test_joined_segments_equal_the_oracle(orc, torch, rows):
    from paper_1810_07806_amd.wcnst import Pool, Solver, split_flags
    d, U = W.random_euler2d(np.random.default_rng(7), 400, 301)
    d.update(bc_x="periodic", bc_y="reflect", gravity=0.5)
    p = orc.problem(d)
    Ro, fo, _ = orc.rhs(p, U, flags=True, nthreads=4)
    r = orc.solve(p, U, cfl=0.5, max_steps=2, nthreads=4)
    assert r["status"] == 0
    s = Solver(d)
    s.set_tuning(rows)
    assert s.stage_shape()["rows1"] == rows
    Ug = s.new_state(U)
    R, fl = s.rhs(Ug, flags=True)
    assert np.array_equal(R.cpu().numpy(), Ro)
    for a, b in zip(split_flags(d, fl.cpu().numpy()), fo):
        assert np.array_equal(a, b)
    s.solve(Ug, cfl=0.5, max_steps=2)
    assert s.status()["t"] == r["t"] and np.array_equal(Ug.cpu().numpy(), r["U"])
    s.close()
    pool = Pool(capacity=2)
    pool.set_tuning(rows)
    V = torch.as_tensor(U).cuda().reshape(-1).clone()
    slot = pool.admit(d, V, torch.empty_like(V), torch.empty_like(V), 1e3, cfl=0.5)
    pool.tick(2)
    assert pool.result(slot)["t"] == r["t"]
    assert np.array_equal(V.cpu().numpy().reshape(U.shape), r["U"])
    pool.close()
