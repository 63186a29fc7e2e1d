"""Members put into cell order from per-cell buckets: more than 8192 cells
(counts summed by cell ranges first), cells that outgrow their bucket by a few
members (chains) and by many (the pass over the keys), several systems, and a
sparse box that keeps the scan / scatter / cell-sort launches.  Every case is
compared with those launches: the same pair lists, and bitwise the same
forces, energies and virials (the same members in the same order)."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


def _crowd(s, seed):
    """Whole molecules moved next to three atoms: 4, 12 and 60 of them, so
    those atoms' cells hold a few, some dozen and more than 64 members beyond
    their buckets."""
    rng = np.random.default_rng(seed)
    pos = s.pos.copy()
    mols = rng.permutation(np.unique(s.mol))
    at = 3
    for target, k in ((mols[0], 4), (mols[1], 12), (mols[2], 60)):
        c = pos[s.mol == target][0]
        for m in mols[at:at + k]:
            sel = s.mol == m
            pos[sel] += c - pos[sel][0] + rng.uniform(0.2, 1.0, 3)
        at += k
    return s.replace(pos=pos)


def _case(name):
    if name == "small":
        return _crowd(w.propane_liquid(1, n_mol=2000), 1)
    if name == "many_cells":
        return w.propane_liquid(2, n_mol=20000)
    if name == "many_cells_crowded":
        return _crowd(w.propane_liquid(3, n_mol=20000), 3)
    if name == "batch":
        return w.replica_batch(4, n_systems=40, min_atoms=1200, max_atoms=3000, total_atoms=90000)
    s = w.propane_liquid(4, n_mol=700)                 # sparse: a liquid in a far larger box
    return s.replace(box=s.box + 150.0)


@pytest.mark.parametrize("name,launches", [("small", 1), ("many_cells", 2), ("many_cells_crowded", 2),
                                           ("batch", 2), ("sparse", 3)])
def test_placement_matches_scan_scatter_sort(monkeypatch, name, launches):
    import torch
    s = _case(name)
    sys_ = s.whole if isinstance(s, w.Batch) else s
    box = s.boxes if isinstance(s, w.Batch) else s.box
    p = torch.from_numpy(sys_.pos).cuda()
    rng = np.random.default_rng(9)
    q = torch.from_numpy(sys_.pos + rng.normal(0.0, 0.4, sys_.pos.shape)).cuda()
    out = {}
    for mode in ("default", "classic"):
        if mode == "classic":
            monkeypatch.setenv("RELRES_PLACE", "classic")
        else:
            monkeypatch.delenv("RELRES_PLACE", raising=False)
        rr = make_relres(sys_, 64)
        if isinstance(s, w.Batch):
            rr.set_systems(s.offsets)
        got = []
        for x in (p, q, p):                            # chains and counts of builds before
            rr.build_lists(x, box)
            got += [t.cpu().numpy() for t in rr.forces(x)]
            got += [rr.pairs(0), rr.pairs(1)]
        assert rr.stats()["place_launches"] == (launches if mode == "default" else 3)
        out[mode] = got
        rr.close()
    for a, b in zip(out["default"], out["classic"]):
        assert np.array_equal(a, b)
