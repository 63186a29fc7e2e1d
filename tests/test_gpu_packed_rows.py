"""Forces-only launches of many small systems, whose rows share waves: systems of
one to a few dozen atoms, some without hybrid atoms, each in its own box, at
automatic and given lane counts, on either side of the rule that chooses the
launch.  Every system against the oracle (FP64 1e-11, FP32 1e-5 of the largest
force) and against the launch with energy and virial, whose waves hold one
system each."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,pair_math", [(64, 0), (32, 32), (32, 64)])
@pytest.mark.parametrize("atoms,lanes", [((1, 4), (0, 0)), ((2, 14), (0, 0)), ((2, 14), (4, 16)),
                                         ((10, 60), (1, 1)), ((10, 60), (16, 64)), ((120, 130), (4, 8))])
def test_small_systems_share_waves(atoms, lanes, precision, pair_math):
    import torch
    rng = np.random.default_rng(atoms[1])
    base = w.two_atoms(5.0)
    systems = []
    for k in range(150):
        n = int(rng.integers(atoms[0], atoms[1] + 1))
        side = int(np.ceil(n ** (1.0 / 3.0)))
        g = np.stack(np.unravel_index(rng.permutation(side ** 3)[:n], (side,) * 3), 1)
        x = 1.0 + 4.2 * g + rng.uniform(-0.4, 0.4, (n, 3))
        hybrid = rng.random(n) < (0.0 if k % 7 == 0 else 0.4)
        systems.append(base.replace(pos=x, types=hybrid.astype(np.int32), mol=np.arange(n, dtype=np.int32),
                                    excl_offsets=np.zeros(n + 1, np.int32),
                                    box=np.array([33.0 + k % 5, 34.0, 35.0 + 0.01 * k])))
    b = w.batch_of(systems)
    print(f"[packed] {b.whole.n} atoms in {len(systems)} systems, lanes {lanes}", flush=True)
    rr = make_relres(b.whole, precision, pair_math)
    rr.set_systems(b.offsets)
    pos = torch.from_numpy(b.whole.pos).cuda()
    rr.build_lists(pos, b.boxes)
    rr.set_launch(*lanes)
    F = rr.forces(pos, want_energy=False, want_virial=False)[0].double().cpu().numpy()
    Fe = rr.forces(pos)[0].double().cpu().numpy()
    want = np.concatenate([oracle.compute(s)[0] for s in systems])
    top = np.abs(want).max()
    tol = 1e-11 if precision == 64 else 1e-5
    assert np.abs(F - want).max() <= tol * top and np.abs(Fe - want).max() <= tol * top
    rr.close()
