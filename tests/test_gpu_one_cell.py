"""A box so close to twice the list radius that its site grid has one cell along
each axis (or along one): members up to a whole box apart in one cell.  Pair
sets bit-exact, with pairs at, just inside and just outside the radii."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, pair_set
from test_gpu_list_filter import _pairs_at

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("other", [32.0 * (1.0 + 5e-11), 50.0])
def test_pairs_in_a_grid_of_one_cell(other):
    import torch
    s = w.two_atoms(5.0)
    edge = 2.0 * (s.rc_out + s.skin) * (1.0 + 5e-11)
    box = np.array([edge, other, other])
    x = _pairs_at((s.rs_out + s.skin, s.rc_out + s.skin), box, 6, seed=4)
    n = len(x)
    s = s.replace(pos=x, box=box, types=np.ones(n, np.int32), mol=np.arange(n, dtype=np.int32),
                  excl_offsets=np.zeros(n + 1, np.int32))
    print(f"[filter] box={box} N={n}", flush=True)
    rr = make_relres(s, 64)
    rr.build_lists(torch.from_numpy(x).cuda(), s.box)
    assert rr.stats()["site_cells"][0] == 1
    for which in (0, 1):
        assert pair_set(rr.pairs(which)) == pair_set(oracle.pairs(s, which))
    rr.close()
