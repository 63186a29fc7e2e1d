"""relres_forces_noalloc with energy and virial at sizes where the automatic
lanes per row decide whether the records fit its static array (16366 blocks):
600000 atoms in rows of about 27 and 97 entries, which fit at 2 and 8 lanes and
not at 4 and 16, and 1.3 million in rows of about 16 and 44, which fit at 1 and
4 and not at 2 and 8.  Same results as relres_forces, bit for bit."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,density,size", [(84, 0.0125, 3), (110, 0.0083, 5)])
def test_large_launches_fit_the_array(side, density, size):
    import torch
    n = side ** 3
    print(f"[noalloc] {n} atoms", flush=True)
    a = density ** (-1.0 / 3.0)
    k = np.arange(n)
    x = (np.stack([k // (side * side), (k // side) % side, k % side], 1) + 0.5) * a
    x += np.random.default_rng(side).normal(scale=0.05, size=x.shape)
    s = w.two_atoms(5.0, box_len=side * a)
    s = s.replace(pos=x, types=(k % size == 0).astype(np.int32), mol=(k // size).astype(np.int32),
                  excl_offsets=np.zeros(n + 1, np.int32))
    rr = make_relres(s, 32)
    p = torch.from_numpy(x).cuda()
    rr.build_lists(p, s.box)
    F, E, W = rr.forces(p)
    F1 = torch.empty_like(F)
    E1 = torch.empty(3, dtype=torch.float64, device="cuda")
    W1 = torch.empty(6, dtype=torch.float64, device="cuda")
    rr.forces_noalloc(p, F1, E1, W1)
    torch.cuda.synchronize()
    assert torch.equal(F, F1) and torch.equal(E, E1) and torch.equal(W, W1)
    rr.close()
