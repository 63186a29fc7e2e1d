"""Dynamics whose list rows outgrow their capacity in the middle of a run: the
run goes on while a build's status is still unread, so it has to return to
that build and repeat the steps after it.  The result must be bitwise that of
a context whose rows were long enough from the start, also when the overflow
is in the run's first or last build, and in several builds of one run."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


def _collapse(side=6, spacing=5.5, box=64.0):
    """A cubic cluster of ordinary atoms in a dilute box (short rows) and the
    velocities of a uniform contraction (long rows later)."""
    g = np.arange(side) - 0.5 * (side - 1)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) * spacing
    x = x + np.random.default_rng(3).normal(scale=0.05, size=x.shape)
    n = len(x)
    s = w.two_atoms(5.0, hybrid=(False, False), box_len=box)
    return s.replace(pos=x + 0.5 * box, types=np.zeros(n, np.int32), mol=np.arange(n, dtype=np.int32),
                     excl_offsets=np.zeros(n + 1, np.int32)), -x * 0.02


def _run(s, v0, steps, grown, every=2):
    import torch
    rr = make_relres(s, 64)
    if grown:                                   # rows sized for the densest frame first
        dense = (s.pos - 32.0) * 0.5 + 32.0
        rr.build_lists(torch.from_numpy(dense).cuda(), s.box)
    p, v = torch.from_numpy(s.pos).cuda(), torch.from_numpy(np.ascontiguousarray(v0)).cuda()
    rr.build_lists(p, s.box)
    rr.set_launch(4, 4)
    rr.md_setup(np.full(s.n, 5000.0), 1.0, 300.0, 1e9, rebuild_every=every)
    before = rr.stats()["regrows"]
    th = rr.md_run(p, v, steps, 1)
    torch.cuda.synchronize()
    out = [t.cpu().numpy() for t in (p, v, th)] + list(rr.md_state())
    regrows = rr.stats()["regrows"] - before
    rr.close()
    return out, regrows


@pytest.mark.parametrize("steps", [24, 13])
def test_overflow_during_a_run(steps):
    s, v = _collapse()
    print(f"[md] collapse N={s.n} steps={steps}", flush=True)
    want, none = _run(s, v, steps, grown=True)
    got, regrows = _run(s, v, steps, grown=False)
    assert none == 0 and regrows >= 1
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


def test_overflow_in_the_first_build_of_a_run():
    """Lists of a dilute frame, then a run from a dense one."""
    import torch
    s, _ = _collapse()
    dense = (s.pos - 32.0) * 0.55 + 32.0
    v0 = np.random.default_rng(4).normal(scale=1e-3, size=dense.shape)
    res = []
    for grown in (True, False):
        rr = make_relres(s, 64)
        rr.set_launch(4, 4)
        rr.build_lists(torch.from_numpy(s.pos).cuda(), s.box)
        p, v = torch.from_numpy(dense).cuda(), torch.from_numpy(v0).cuda()
        if grown:
            rr.build_lists(p, s.box)
        rr.md_setup(np.full(s.n, 5000.0), 1.0, 300.0, 1e9, rebuild_every=3)
        th = rr.md_run(p, v, 8, 2)
        torch.cuda.synchronize()
        res.append([t.cpu().numpy() for t in (p, v, th)])
        rr.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)
