"""Lane counts of several systems may change wherever they could with one: the
wave tables of every lane count are there from relres_set_systems on, so a
change allocates nothing, leaves captured launches valid and works inside a
capture."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu

LANES = [(1, 1), (2, 8), (4, 16), (16, 4), (32, 64), (64, 2)]


def _batch():
    import torch
    b = w.replica_batch(1, n_systems=5, min_atoms=300, max_atoms=900, total_atoms=3000)
    rr = make_relres(b.whole, 64)
    rr.set_systems(b.offsets)
    pos = torch.from_numpy(b.whole.pos).cuda()
    rr.build_lists(pos, b.boxes)
    rr.set_launch(64, 64)                       # the largest buffers once
    rr.forces(pos)
    return b, rr, pos


def _forces(rr, pos, out=None):
    return rr.forces(pos, out=out, want_energy=False, want_virial=False)[0]


def test_lane_changes_leave_captured_launches_valid():
    b, rr, pos = _batch()
    before = rr.generation()
    for lanes in LANES:
        print(f"[lanes] {lanes}", flush=True)
        rr.set_launch(*lanes)
        _forces(rr, pos)
        rr.forces(pos)
    rr.set_launch(0, 0)
    rr.stats()
    _forces(rr, pos)
    assert rr.generation() == before
    rr.close()


def test_lane_changes_inside_a_capture():
    import torch
    b, rr, pos = _batch()
    want = {}
    for lanes in LANES:
        rr.set_launch(*lanes)
        want[lanes] = _forces(rr, pos).clone()
    torch.cuda.synchronize()
    rr.close()
    b, rr, pos = _batch()
    outs = {lanes: torch.zeros_like(want[lanes]) for lanes in LANES}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print("[lanes] capture", flush=True)
    with torch.cuda.graph(graph):
        for lanes in LANES:
            rr.set_launch(*lanes)
            _forces(rr, pos, outs[lanes])
    for replay in range(3):
        for o in outs.values():
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for lanes in LANES:
            assert torch.equal(outs[lanes], want[lanes]), (replay, lanes)
    rr.close()


@pytest.mark.parametrize("side", [40, 84])
@pytest.mark.parametrize("energy_first", [False, True])
def test_either_kind_of_call_prepares_the_other(side, energy_first):
    """Forces-only launches and launches with energy and virial split their rows
    differently (64000 and 592704 atoms): a call of one kind leaves nothing for
    the first of the other to allocate, so that one may be captured and the
    other's captured launches stay valid."""
    import torch
    n, density = side ** 3, 0.0125
    print(f"[lanes] {n} atoms, energy first {energy_first}", flush=True)
    a = density ** (-1.0 / 3.0)
    k = np.arange(n)
    x = (np.stack([k // (side * side), (k // side) % side, k % side], 1) + 0.5) * a
    s = w.two_atoms(5.0, box_len=side * a)
    s = s.replace(pos=x, types=(k % 3 == 0).astype(np.int32), mol=(k // 3).astype(np.int32),
                  excl_offsets=np.zeros(n + 1, np.int32))
    rr = make_relres(s, 32)
    p = torch.from_numpy(x).cuda()
    rr.build_lists(p, s.box)
    rr.forces(p, want_energy=energy_first, want_virial=energy_first)
    before = rr.generation()
    rr.forces(p, want_energy=not energy_first, want_virial=not energy_first)
    torch.cuda.synchronize()
    assert rr.generation() == before
    rr.close()
