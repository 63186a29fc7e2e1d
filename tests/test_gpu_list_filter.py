"""The list kernel's FP32 distance filter and its exclusion tests.

The kernel decides a pair by an FP32 distance unless that lies within its
rounding bound of the list radius, where the FP64 membership recipe decides;
pair sets must be the oracle's (bit-exact) for pairs at, just inside and just
outside the radius.  Boxes: few cells per axis (differences folded to the
nearest image) and enough that they need not be, cubic and not; both
candidate counts.  Exclusions: an index range around the atom (chains), a
scattered list, both with and without the same-molecule rule."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, pair_set

pytestmark = pytest.mark.gpu

# relative offsets from the list radius: rounding level, far below the
# filter's bound (about 1e-6), around it and past it
OFFSETS = np.array([0.0, 1e-16, 3e-16, 1e-15, 1e-13, 1e-10, 1e-8, 3e-7, 1e-6, 3e-6, 1e-5, 1e-4])


def _pairs_at(radii, box, per, seed):
    """Pairs of atoms at radius * (1 +- offset), anywhere in the box."""
    rng = np.random.default_rng(seed)
    x = []
    for r in radii:
        for eps in np.concatenate([OFFSETS, -OFFSETS]):
            a = rng.uniform(0.0, 1.0, size=(per, 3)) * box
            u = rng.normal(size=(per, 3))
            u[0] = [1.0, 0.0, 0.0]           # one along an axis
            u /= np.linalg.norm(u, axis=1, keepdims=True)
            x += [a, a + r * (1.0 + eps) * u]
    return w.wrap(np.concatenate(x), np.asarray(box, float))


@pytest.mark.parametrize("cand", [2, 4])
@pytest.mark.parametrize("box", [(33.0, 33.0, 33.0), (41.0, 70.0, 36.0), (90.0, 85.0, 97.0)])
def test_pairs_at_the_list_radius(box, cand):
    import torch
    s = w.two_atoms(5.0)
    x = _pairs_at((s.rs_out + s.skin, s.rc_out + s.skin), np.array(box), 6, seed=3)
    n = len(x)
    s = s.replace(pos=x, box=np.array(box), types=np.ones(n, np.int32),
                  mol=np.arange(n, dtype=np.int32), excl_offsets=np.zeros(n + 1, np.int32))
    print(f"[filter] box={box} cand={cand} N={n}", flush=True)
    rr = make_relres(s, 64)
    rr.set_list_launch(0, 0, cand)
    rr.build_lists(torch.from_numpy(x).cuda(), s.box)
    for which in (0, 1):
        assert pair_set(rr.pairs(which)) == pair_set(oracle.pairs(s, which))
    rr.close()


@pytest.mark.parametrize("same_mol", [False, True])
@pytest.mark.parametrize("kind", ["range", "scattered"])
def test_exclusion_ranges_and_lists(kind, same_mol):
    """Atoms whose exclusions fill an index range with the atom itself (1 to
    6 partners: chain ends and middles) or do not, in one system."""
    import torch
    s = w.random_molecules(21, 140, 35.0, kind="propane", min_dist=2.2)
    n = s.n
    rng = np.random.default_rng(5)
    if kind == "range":
        part = [[j for j in range(max(0, i - 3), min(n, i + 4)) if j != i] for i in range(n)]
    else:
        part = [sorted(set(rng.integers(0, n, size=rng.integers(0, 9)).tolist()) - {i})
                for i in range(n)]
    off = np.concatenate([[0], np.cumsum([len(p) for p in part])]).astype(np.int32)
    s = s.replace(excl_offsets=off, excl_idx=np.array([j for p in part for j in p], np.int32),
                  exclude_same_mol=same_mol, types=np.ones(n, np.int32))
    print(f"[filter] exclusions {kind} same_mol={same_mol}", flush=True)
    rr = make_relres(s, 64)
    rr.build_lists(torch.from_numpy(s.pos).cuda(), s.box)
    for which in (0, 1):
        assert pair_set(rr.pairs(which)) == pair_set(oracle.pairs(s, which))
    rr.close()
