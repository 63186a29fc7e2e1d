"""Non-finite positions are reported by every build that sees them, not only by
the first of a context: one atom, a whole wave and all atoms, with good builds
between, waited for or not, one system or several."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("systems", [1, 2])
@pytest.mark.parametrize("wait", [True, False])
def test_every_bad_build_is_refused(wait, systems):
    import torch
    from paper_2104_10231_amd.relres import RelResError
    s = w.random_molecules(seed=11, n_mol=120, box_len=34.0, kind="propane", min_dist=2.9,
                           hybrid_fraction=0.9)
    rr = make_relres(s)
    box = s.box
    if systems == 2:
        rr.set_systems(np.array([0, s.n // 2, s.n], np.int32))
        box = np.stack([s.box, s.box])
    good = torch.from_numpy(s.pos).cuda()
    rr.build_lists(good, box)
    F = rr.forces(good, want_energy=False, want_virial=False)[0].clone()
    for lo, hi, what in ((5, 6, "nan"), (64, 128, "inf"), (0, s.n, "-inf"), (s.n - 1, s.n, "nan")):
        print(f"[nonfinite] atoms {lo}..{hi} {what} wait {wait} systems {systems}", flush=True)
        bad = good.clone()
        bad[lo:hi, 1] = float(what)
        with pytest.raises(RelResError) as e:
            rr.build_lists(bad, box, wait=wait)
            if not wait:
                rr.check_lists()
        assert "non-finite" in str(e.value)
        rr.build_lists(good, box)
        assert torch.equal(rr.forces(good, want_energy=False, want_virial=False)[0], F)
    rr.close()
