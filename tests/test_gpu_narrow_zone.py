"""A switching zone at r_s of zero width, of one unit in the last place and of
a few: the polynomial's coefficients grow as the cube of its reciprocal width,
past FP32's range, and must not reach the constant part inside it (hybrid pairs
below r_s-).  Forces and energies against the oracle, at the parity bars of the
precision (FP64 1e-11, FP32 1e-5 relative RMS; energies 1e-12 and 1e-7)."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,pair_math", [(64, 0), (32, 32), (32, 64)])
@pytest.mark.parametrize("ulps", [0, 1, 20])
def test_zone_of_a_few_units_in_the_last_place(ulps, precision, pair_math):
    import torch
    rs = 5.75
    s = w.random_molecules(seed=12, n_mol=150, box_len=34.0, kind="propane", min_dist=2.9,
                           hybrid_fraction=0.9).replace(rs_in=rs, rs_out=rs + ulps * np.spacing(rs))
    print(f"[zone] {ulps} ulps precision={precision} pair_math={pair_math}", flush=True)
    Fr, Er, _ = oracle.compute(s)
    rr = make_relres(s, precision, pair_math)
    p = torch.from_numpy(s.pos).cuda()
    rr.build_lists(p, s.box)
    F0 = rr.forces(p, want_energy=False, want_virial=False)[0].double().cpu().numpy()
    F, E, _ = rr.forces(p)
    F, E = F.double().cpu().numpy(), E.cpu().numpy()
    ftol, etol = (1e-11, 1e-12) if precision == 64 else (1e-5, 1e-7)
    assert rel_rms(F0, Fr) <= ftol and rel_rms(F, Fr) <= ftol
    assert abs(E[0] - Er[0]) <= etol * np.abs(Er).max()
    rr.close()
