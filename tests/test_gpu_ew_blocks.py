"""Energy and virial of launches of few blocks: up to 128 one block waits for
all the others, above that in groups; from 8 blocks to 160 and both sides of
the limit, against the oracle at the FP64 bar used elsewhere (1e-12 of the
energy and of the largest virial component), repeated calls bitwise equal."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mol,lanes", [(2, (1, 1)), (500, (2, 2)), (500, (4, 4)), (500, (8, 8)),
                                         (500, (16, 16)), (500, (16, 32)), (520, (16, 16))])
def test_energy_and_virial_of_few_blocks(n_mol, lanes):
    import torch
    s = w.propane_liquid(2, n_mol=max(n_mol, 500))
    if n_mol == 2:
        keep = s.mol < 2
        s = s.replace(pos=s.pos[keep], types=s.types[keep], mol=s.mol[keep],
                      excl_offsets=np.zeros(int(keep.sum()) + 1, np.int32), excl_idx=np.zeros(0, np.int32))
    print(f"[ew] N={s.n} lanes={lanes}", flush=True)
    rr = make_relres(s, 64)
    rr.set_launch(*lanes)
    p = torch.from_numpy(np.ascontiguousarray(s.pos)).cuda()
    rr.build_lists(p, s.box)
    F, E, W = rr.forces(p)
    for _ in range(3):
        F2, E2, W2 = rr.forces(p)
        assert torch.equal(F, F2) and torch.equal(E, E2) and torch.equal(W, W2)
    rr.sync()
    Fr, Er, Wr = oracle.compute(s)
    assert rel_rms(F.cpu().numpy(), Fr) <= 1e-11
    assert abs(E[0].item() - Er[0]) <= 1e-12 * max(abs(Er[0]), 1e-300)
    assert np.abs(W.cpu().numpy() - Wr).max() <= 1e-12 * max(np.abs(Wr).max(), 1e-300)
    rr.close()
