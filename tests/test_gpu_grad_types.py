"""The adjoint kernel at every bound on the number of types it is built for
(2, 4 and 8, exactly and below) and at the smallest and largest lane splits:
packed tables of one to 64 type pairs, rows longer and shorter than a round
of two entries per lane, a block partial per bin.  Bars as in
test_gpu_grad.py: norm-relative 1e-9 for positions, 1e-8 per parameter."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes", [(1, 1), (32, 64)])
@pytest.mark.parametrize("ntypes", [1, 2, 3, 5, 8])
def test_types_and_lane_splits(ntypes, lanes):
    import torch
    s = w.random_molecules(31 + ntypes, 110, 34.0, kind="propane", min_dist=2.9)
    rng = np.random.default_rng(ntypes)
    hybrid = rng.uniform(size=ntypes) < 0.6
    hybrid[-1] = True
    s = s.replace(types=rng.integers(0, ntypes, size=s.n).astype(np.int32),
                  eps_fg=rng.uniform(0.05, 0.3, ntypes), sig_fg=rng.uniform(3.4, 4.0, ntypes),
                  eps_cg=np.where(hybrid, rng.uniform(1, 3, ntypes), 0.0),
                  sig_cg=rng.uniform(4.0, 4.8, ntypes))
    print(f"[grad] ntypes={ntypes} lanes={lanes} N={s.n}", flush=True)
    g, e_bar = rng.normal(size=(s.n, 3)), 0.8
    rr = make_relres(s, 64)
    rr.set_launch(*lanes)
    pos = torch.from_numpy(s.pos).cuda()
    rr.build_lists(pos, s.box)
    up = torch.from_numpy(g).cuda()
    eb = torch.full((1,), e_bar, dtype=torch.float64, device="cuda")
    dp, dt = (t.cpu().numpy() for t in rr.backward_types(pos, up, eb))
    again = rr.backward_types(pos, up, eb)
    assert np.array_equal(again[0].cpu().numpy(), dp) and np.array_equal(again[1].cpu().numpy(), dt)
    dt_ref, dp_ref = oracle.grad(s, g, e_bar)
    assert np.linalg.norm(dp - dp_ref) <= 1e-9 * np.linalg.norm(dp_ref)
    scale = np.abs(dt_ref).max()
    assert np.all(np.abs(dt - dt_ref) <= 1e-8 * np.abs(dt_ref) + 1e-10 * scale), (dt, dt_ref)
    rr.close()
