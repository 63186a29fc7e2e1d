"""What a dynamics run checks of its list builds although it does not wait for
them: displacements past half the skin in every stretch of steps between two
builds and after the last, also where rows overflowed."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres
from test_gpu_md import _ctx, _hexane
from test_gpu_md_regrow import _collapse

pytestmark = pytest.mark.gpu


def _stale(call):
    from paper_2104_10231_amd.relres import RelResError, RELRES_ERR_STALE_LISTS
    with pytest.raises(RelResError) as e:
        call()
    assert e.value.code == RELRES_ERR_STALE_LISTS


@pytest.mark.parametrize("steps,skin", [(1, 2e-4), (39, 0.05), (41, 0.05)])
def test_steps_without_a_build_are_checked(steps, skin):
    """Builds every 40 steps and a skin outrun within one step (atoms move some
    7e-3 A a step) or within 39; two runs in a row, one step past a build too."""
    import torch
    s = _hexane(n_mol=60, seed=5).replace(skin=skin)
    print(f"[md] stale lists, {steps} steps", flush=True)
    rr, p = _ctx(s)
    v = torch.from_numpy(np.ascontiguousarray(s.bonded["velocities"])).cuda()
    rr.md_setup(s.bonded["masses"], 1.0, 300.0, 100.0, rebuild_every=40)
    for _ in range(2):
        _stale(lambda: rr.md_run(p, v, steps))
    rr.close()


def _caged(oscillator):
    """A light atom, near a corner of its cell, between six heavy ones whose
    forces on it cancel, and a shell of heavy atoms that enters its list radius
    (8 A, beyond the 6 A of the forces) within ten steps: its row then outgrows
    its capacity, and what is stored of it pushes it past half the skin (1 A) in
    nine steps.  With `oscillator` also a bonded pair far from everything,
    released from 1.4 A of stretch: each atom moves 0.7 A in the first ten steps,
    then 1.27 A in nine and 1.4 A in ten (60 degrees of its period each ten)."""
    i = np.arange(100) + 0.5
    z, phi = 1.0 - 2.0 * i / 100, np.pi * (1.0 + 5.0 ** 0.5) * i
    q = np.sqrt(1.0 - z * z)
    shell = np.stack([q * np.cos(phi), q * np.sin(phi), z], 1)
    x = np.vstack([np.zeros((1, 3)), 3.2 * np.eye(3), -3.2 * np.eye(3), 8.3 * shell]) + [37.0, 37.3, 37.7]
    v = np.vstack([np.zeros((7, 3)), -0.05 * shell])
    mass = np.full(len(x), 1e7)
    mass[0] = 0.1
    if oscillator:
        x = np.vstack([x, [[5.0, 5.0, 5.0], [5.0 + 12.0 + 2.8, 5.0, 5.0]]])
        v = np.vstack([v, np.zeros((2, 3))])
        mass = np.append(mass, [100.0, 100.0])
    n = len(x)
    s = w.two_atoms(5.0, hybrid=(False, False), box_len=64.0)
    s = s.replace(pos=x, types=np.zeros(n, np.int32), mol=np.arange(n, dtype=np.int32),
                  excl_offsets=np.zeros(n + 1, np.int32))
    none = np.zeros((0, 4), np.int32)
    bonded = dict(bonds=np.zeros((0, 2), np.int32), bond_k=np.zeros(0), bond_r0=np.zeros(0),
                  angles=none[:, :3], angle_k=np.zeros(0), angle_t0=np.zeros(0), dihedrals=none,
                  dih_k=np.zeros(0), dih_n=np.zeros(0, np.int32), dih_d=np.zeros(0),
                  pairs14=none[:, :2], scale14=0.0)
    if oscillator:
        omega = np.pi / 30.0
        bonded.update(bonds=np.array([[n - 2, n - 1]], np.int32), bond_r0=np.array([12.0]),
                      bond_k=np.array([omega * omega * 100.0 / (4.0 * 4.184e-4)]))
    return s, v, mass, bonded


@pytest.mark.parametrize("steps", [19, 25])
@pytest.mark.parametrize("oscillator", [False, True])
def test_steps_after_an_overflowed_build(oscillator, steps):
    """The steps after an overflowed build (the run's last, or the one before)
    are repeated whatever they did, and their repetition is checked: the run ends
    as one whose rows were long enough from the start, with its result or with
    its error."""
    import torch
    s, v0, mass, bonded = _caged(oscillator)
    print(f"[md] overflow at step 10 of {steps}, oscillator {oscillator}", flush=True)
    res = []
    for grown in (True, False):
        rr = make_relres(s, 64)
        rr.set_bonded(bonded)
        p, v = torch.from_numpy(s.pos).cuda(), torch.from_numpy(v0).cuda()
        if grown:                               # rows sized for the contracted shell
            rr.build_lists(p + 10.0 * v, s.box)
        rr.build_lists(p, s.box)
        rr.set_launch(4, 4)
        rr.md_setup(mass, 1.0, 300.0, 1e9, rebuild_every=10)
        before = rr.stats()["regrows"]
        if oscillator:
            _stale(lambda: rr.md_run(p, v, steps))
        else:
            rr.md_run(p, v, steps)
        torch.cuda.synchronize()
        res.append((p.cpu().numpy(), v.cpu().numpy(), rr.stats()["regrows"] - before))
        rr.close()
    assert res[0][2] == 0 and res[1][2] >= 1
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


def _bits(t):
    return t.cpu().numpy().view(np.int64)


@pytest.mark.parametrize("steps", [3, 25])
def test_nonfinite_positions_leave_the_run_untouched(steps):
    """Refused by the first build's status, which is read after steps were
    enqueued behind it: positions, velocities and thermostat are the caller's."""
    import torch
    from paper_2104_10231_amd.relres import RelResError
    s = _hexane(n_mol=80, seed=5)
    print(f"[md] non-finite position, {steps} steps", flush=True)
    rr, p = _ctx(s)
    rr.md_setup(s.bonded["masses"], 1.0, 300.0, 100.0, rebuild_every=10)
    rr.md_state(1e-4, 2e-3)
    p[17, 1] = float("nan")
    v = torch.from_numpy(np.ascontiguousarray(s.bonded["velocities"])).cuda()
    before = _bits(p), _bits(v)
    with pytest.raises(RelResError) as e:
        rr.md_run(p, v, steps)
    assert "non-finite" in str(e.value)
    assert np.array_equal(_bits(p), before[0]) and np.array_equal(_bits(v), before[1])
    assert rr.md_state() == (1e-4, 2e-3)
    rr.close()


def test_stale_lists_leave_the_build_that_found_them():
    """Atoms outrun the skin in the first five steps: with builds every five, a
    run of 20 steps ends where the build at step five found it, as a run of
    five does."""
    import torch
    s = _hexane(n_mol=60, seed=5).replace(skin=0.02)
    res = []
    for steps in (5, 20):
        print(f"[md] stale at step 5 of {steps}", flush=True)
        rr, p = _ctx(s)
        v = torch.from_numpy(np.ascontiguousarray(s.bonded["velocities"])).cuda()
        rr.md_setup(s.bonded["masses"], 1.0, 300.0, 100.0, rebuild_every=5)
        _stale(lambda: rr.md_run(p, v, steps))
        res.append(_bits(p))
        rr.close()
    assert np.array_equal(*res)


@pytest.mark.parametrize("steps", [1, 25])
def test_a_run_that_blows_up_is_reported(steps):
    """A velocity that is no number: the atom's positions after the first step
    are none either, before any build could see them (builds every 40)."""
    import torch
    s = _hexane(n_mol=80, seed=5)
    print(f"[md] velocity NaN, {steps} steps", flush=True)
    rr, p = _ctx(s)
    rr.md_setup(s.bonded["masses"], 1.0, 300.0, 1e9, rebuild_every=40)
    v = torch.from_numpy(np.ascontiguousarray(s.bonded["velocities"])).cuda()
    v[s.n - 1, 2] = float("nan")
    _stale(lambda: rr.md_run(p, v, steps))
    rr.close()


def test_overflow_in_the_first_build_goes_back_to_it():
    """Lists of a dilute frame, then a run from a dense one, whose first build
    overflows, against a run whose rows were sized for the dense frame: the same
    result bit for bit, with and without a return to the build."""
    import torch
    s, _ = _collapse()
    dense = (s.pos - 32.0) * 0.55 + 32.0
    v0 = np.random.default_rng(4).normal(scale=1e-3, size=dense.shape)
    res, regrows = [], []
    for grown in (True, False):
        print(f"[md] first build, grown {grown}", flush=True)
        rr = make_relres(s, 64)
        rr.set_launch(4, 4)
        rr.build_lists(torch.from_numpy(s.pos).cuda(), s.box)
        p, v = torch.from_numpy(dense).cuda(), torch.from_numpy(v0).cuda()
        if grown:
            rr.build_lists(p, s.box)
        rr.md_setup(np.full(s.n, 5000.0), 1.0, 300.0, 1e9, rebuild_every=3)
        before = rr.stats()["regrows"]
        th = rr.md_run(p, v, 8, 2)
        torch.cuda.synchronize()
        regrows.append(rr.stats()["regrows"] - before)
        res.append([t.cpu().numpy() for t in (p, v, th)])
        rr.close()
    assert regrows[0] == 0 and regrows[1] >= 1
    for a, b in zip(*res):
        assert np.array_equal(a, b)
