"""One-launch placement of cells far beyond their bucket: 8 to 1300 atoms in a
ball of 2 A (a cell's bucket, the chains beyond it, the most that a wave ranks,
more than that), in grids of few cells and of more than 8192, and a dense slab
in an empty box, where many cells outgrow buckets sized for the mean.  Each
against the scan / scatter / cell-sort launches: the same pair lists, and
bitwise the same forces, energies and virials."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu

BALLS = (8, 16, 17, 24, 40, 63, 64, 65, 80, 81, 100, 128, 129, 200, 300, 1023, 1024, 1025, 1300)


def _balls(box, n_gas, seed):
    rng = np.random.default_rng(seed)
    k = int(np.ceil(len(BALLS) ** (1.0 / 3.0)))
    at = (np.stack(np.unravel_index(np.arange(len(BALLS)), (k,) * 3), 1) + 0.5) * (box / k)
    x = [rng.uniform(0.0, box, (n_gas, 3))]
    for c, m in zip(at, BALLS):
        u = rng.normal(size=(m, 3))
        x.append(c + 2.0 * u / np.linalg.norm(u, axis=1)[:, None] * rng.random((m, 1)) ** (1.0 / 3.0))
    x = np.concatenate(x)
    return x[rng.permutation(len(x))], np.full(3, box)


def _slab():
    rng = np.random.default_rng(5)
    side, a = 30, 0.02 ** (-1.0 / 3.0)
    k = np.arange(side ** 3)
    x = (np.stack([k // side ** 2, (k // side) % side, k % side], 1) + 0.5) * a
    x = x + rng.normal(scale=0.1, size=x.shape)
    return x[rng.permutation(len(x))], np.array([side * a, side * a, 10.0 * side * a])


@pytest.mark.parametrize("name,launches", [("few_cells", 1), ("many_cells", 2), ("slab", 2)])
@pytest.mark.parametrize("hybrid", [1.0, 0.4])
def test_crowded_cells_match_scan_scatter_sort(monkeypatch, name, launches, hybrid):
    import torch
    x, box = {"few_cells": lambda: _balls(130.0, 3000, 1), "many_cells": lambda: _balls(180.0, 20000, 2),
              "slab": _slab}[name]()
    n = len(x)
    rng = np.random.default_rng(3)
    s = w.two_atoms(5.0).replace(pos=x, box=box, types=(rng.random(n) < hybrid).astype(np.int32),
                                 mol=np.arange(n, dtype=np.int32), excl_offsets=np.zeros(n + 1, np.int32))
    print(f"[crowded] {name} N={n}", flush=True)
    p = torch.from_numpy(x).cuda()
    q = p + 0.3 * torch.randn(p.shape, dtype=p.dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    out = {}
    for mode in ("default", "classic"):
        if mode == "classic":
            monkeypatch.setenv("RELRES_PLACE", "classic")
        else:
            monkeypatch.delenv("RELRES_PLACE", raising=False)
        rr = make_relres(s, 64)
        got = []
        for y in (p, q, p):
            rr.build_lists(y, box)
            got += [t.cpu().numpy() for t in rr.forces(y)]
            got += [rr.pairs(0), rr.pairs(1)]
        assert rr.stats()["place_launches"] == (launches if mode == "default" else 3)
        out[mode] = got
        rr.close()
    for a, b in zip(out["default"], out["classic"]):
        assert np.array_equal(a, b)
