"""Force launches of several systems: every wave holds rows of one system, so
systems whose rows do not fill their last wave, systems of a few molecules, of
none, and without hybrid atoms meet every lane count.  Forces, energies and
virials of each against the oracle, with and without energy/virial, and the
same after the lanes change under lists already built.  Bars: FP64 forces
1e-11 relative RMS, energies and virials 1e-12."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, rel_rms

pytestmark = pytest.mark.gpu


def _batch():
    s = [w.random_molecules(40 + k, n, 33.0 + k, kind="propane", min_dist=2.9, hybrid_fraction=h)
         for k, (n, h) in enumerate(((61, 0.8), (1, 1.0), (0, 0.0), (43, 0.0), (90, 0.5), (2, 0.0)))]
    s[2] = s[0].replace(pos=np.zeros((0, 3)), types=np.zeros(0, np.int32), mol=np.zeros(0, np.int32),
                        excl_offsets=np.zeros(1, np.int32), box=np.full(3, 35.0))
    return w.batch_of(s)


@pytest.mark.parametrize("lanes", [(0, 0), (1, 1), (2, 8), (16, 32), (64, 64)])
def test_uneven_systems_at_every_lane_count(lanes):
    import torch
    b = _batch()
    print(f"[batch] sizes={np.diff(b.offsets).tolist()} lanes={lanes}", flush=True)
    rr = make_relres(b.whole, 64)
    rr.set_systems(b.offsets)
    pos = torch.from_numpy(b.whole.pos).cuda()
    rr.build_lists(pos, b.boxes)
    rr.set_launch(*lanes)
    F, E, W = rr.forces(pos)
    F2 = rr.forces(pos, want_energy=False, want_virial=False)[0]
    torch.cuda.synchronize()
    F, F2, E, W = (t.cpu().numpy() for t in (F, F2, E, W))
    for k, s in enumerate(b.systems):
        sl = slice(int(b.offsets[k]), int(b.offsets[k + 1]))
        if s.n == 0:
            assert np.all(E[k] == 0.0) and np.all(W[k] == 0.0)
            continue
        Fr, Er, Wr = oracle.compute(s)
        for got in (F[sl], F2[sl]):
            if np.any(Fr):
                assert rel_rms(got, Fr) <= 1e-11, k
            else:
                assert np.all(got == 0.0)
        assert abs(E[k, 0] - Er[0]) <= 1e-12 * max(abs(Er[0]), abs(Er[1]), 1e-300)
        assert np.abs(W[k] - Wr).max() <= 1e-12 * max(np.abs(Wr).max(), 1e-300)
    rr.close()
