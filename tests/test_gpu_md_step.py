"""The dynamics step's launches: drift and bonded forces in one launch where no
term crosses a bonded block, in two where one does, and the half kick in the
force launch at every number of lanes per row.

Both forms of a system do the same arithmetic (a bond of zero strength across
the blocks selects the second), up to how the compiler contracts it, so FP64
runs of 20 steps agree to 1e-11 of the largest velocity and FP32 ones, whose
bonded forces are rounded to FP32, to 1e-5.  Lanes change the order of a row's
sum: an FP64 force of ~200 terms differs by at most 200 x 1.1e-16 x its sum of
magnitudes (below 1e3 x the force), 2e-11 of it, an FP32 one by 1e-2 x 1e-2 of
it in the same way, and a step changes a velocity by less than itself."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres
from test_gpu_md_regrow import _collapse

pytestmark = pytest.mark.gpu


def _run(s, bonded, precision, steps, every=5, thermo=5, lanes=None, start=None, dense=None, v0=None,
         tau=100.0):
    import torch
    rr = make_relres(s, precision)
    rr.set_bonded(bonded)
    if dense is not None:
        rr.build_lists(torch.from_numpy(dense).cuda(), s.box)
    p = torch.from_numpy(np.ascontiguousarray(s.pos)).cuda()
    v = torch.from_numpy(np.ascontiguousarray(bonded["velocities"] if v0 is None else v0)).cuda()
    rr.build_lists(p, s.box)
    if lanes is not None:
        rr.set_launch(*lanes)
    rr.md_setup(bonded["masses"], 1.0, 300.0, tau, rebuild_every=every)
    before = rr.stats()["regrows"]
    th = rr.md_run(p, v, steps, thermo)
    torch.cuda.synchronize()
    regrows = rr.stats()["regrows"] - before
    out = [t.cpu().numpy() for t in (p, v, th)] + [np.array(rr.md_state())]
    rr.close()
    return out, regrows


def _crossing(bonded, n):
    """The same terms and a bond of zero strength from the first to the last atom."""
    b = dict(bonded)
    b["bonds"] = np.concatenate([np.asarray(b["bonds"], np.int32).reshape(-1, 2),
                                 np.array([[0, n - 1]], np.int32)])
    b["bond_k"] = np.append(b["bond_k"], 0.0)
    b["bond_r0"] = np.append(b["bond_r0"], 1.0)
    return b


def _many_passes(s, seed):
    """Terms within clusters of 30 atoms, more than one pass of force slots."""
    rng = np.random.default_rng(seed)
    b = dict(s.bonded)
    clusters = s.n // 30
    pick = lambda k, m: np.concatenate([30 * c + np.stack([rng.choice(30, k, replace=False)    # noqa: E731
                                        for _ in range(m)]) for c in range(clusters)]).astype(np.int32)
    b["bonds"], b["angles"], b["dihedrals"], b["pairs14"] = pick(2, 500), pick(3, 300), pick(4, 300), pick(2, 10)
    for key, name in (("bonds", "bond"), ("angles", "angle"), ("dihedrals", "dih")):
        b[name + "_k"] = rng.uniform(1e-3, 3e-3, len(b[key]))
    b["bond_r0"] = rng.uniform(5.0, 20.0, len(b["bonds"]))
    b["angle_t0"] = rng.uniform(1.0, 2.0, len(b["angles"]))
    b["dih_n"] = rng.integers(0, 5, len(b["dihedrals"])).astype(np.int32)
    b["dih_d"] = rng.uniform(0.0, 3.0, len(b["dihedrals"]))
    b["scale14"] = 0.0
    return b


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("passes", ["one", "many"])
def test_one_and_two_launch_steps_agree(passes, precision):
    s = w.hexane_liquid(3, n_mol=150, density=0.012)
    if passes == "many":
        # random angles of exact zigzag chains would hold collinear triplets,
        # where the force on an angle is not finite (the oracle's neither)
        s = s.replace(pos=s.pos + np.random.default_rng(6).normal(0.0, 0.1, s.pos.shape))
    b = s.bonded if passes == "one" else _many_passes(s, 4)
    print(f"[md] step launches N={s.n} passes={passes} precision={precision}", flush=True)
    (x, v, th, st), _ = _run(s, b, precision, 20)
    (x2, v2, th2, st2), _ = _run(s, _crossing(b, s.n), precision, 20)
    tol = 1e-11 if precision == 64 else 1e-5
    assert np.isfinite(v).all() and np.abs(v).max() > 0
    assert np.abs(v - v2).max() <= tol * np.abs(v).max()
    assert np.abs(x - x2).max() <= 20.0 * tol * np.abs(v).max()
    assert np.abs(th - th2).max() <= tol * np.abs(th).max()
    assert np.abs(st - st2).max() <= max(tol * np.abs(st).max(), 1e-300)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("lanes", [(1, 1), (2, 1), (4, 2), (64, 32)])
def test_half_kick_at_every_lane_count(lanes, precision):
    s = w.hexane_liquid(5, n_mol=150, density=0.012)
    print(f"[md] half kick lanes={lanes} precision={precision}", flush=True)
    (x, v, th, _), _ = _run(s, s.bonded, precision, 4, every=2, thermo=2, lanes=(8, 8))
    (x2, v2, th2, _), _ = _run(s, s.bonded, precision, 4, every=2, thermo=2, lanes=lanes)
    tol = 1e-10 if precision == 64 else 1e-4
    assert np.abs(v - v2).max() <= tol * np.abs(v).max()
    assert np.abs(x - x2).max() <= 4.0 * tol * np.abs(v).max()
    assert np.abs(th - th2).max() <= tol * np.abs(th).max()


@pytest.mark.parametrize("crossing", [False, True])
def test_overflow_with_bonded_terms(crossing):
    """A run that goes back to a build repeats that step's bonded forces too."""
    s, v0 = _collapse()
    n = s.n
    b = dict(bonds=np.arange(n, dtype=np.int32).reshape(-1, 2), bond_k=np.full(n // 2, 5.0),
             bond_r0=np.full(n // 2, 4.0), angles=np.zeros((0, 3), np.int32), angle_k=np.zeros(0),
             angle_t0=np.zeros(0), dihedrals=np.zeros((0, 4), np.int32), dih_k=np.zeros(0),
             dih_n=np.zeros(0, np.int32), dih_d=np.zeros(0), pairs14=np.zeros((0, 2), np.int32),
             scale14=0.0, masses=np.full(n, 5000.0))
    if crossing:
        b = _crossing(b, n)
    dense = (s.pos - 32.0) * 0.5 + 32.0
    want, none = _run(s, b, 64, 24, every=2, thermo=1, lanes=(4, 4), dense=dense, v0=v0, tau=1e9)
    got, regrows = _run(s, b, 64, 24, every=2, thermo=1, lanes=(4, 4), v0=v0, tau=1e9)
    assert none == 0 and regrows >= 1
    for a, c in zip(got, want):
        assert np.array_equal(a, c)
