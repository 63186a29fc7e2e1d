"""Kinetic energies of dynamics runs whose force launches leave few partial sums
(read by the drift directly) and many (added up in groups before): the kinetic
energy put out is that of the velocities, and both give the same trajectory.

592704 atoms; a sum of 3 n products in any order is within 3 n 2^-53 = 2e-10 of
the exact one, relative to it, and so are two of them; the thermostat's share of
a velocity is far below 1, and forces of rows of ~130 entries differ by less
than 1e-11 of theirs."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu

FTM2V = 4.184e-4


def test_few_and_many_partials_agree():
    import torch
    side, density = 84, 0.0125
    n = side ** 3
    a = density ** (-1.0 / 3.0)
    k = np.arange(n)
    rng = np.random.default_rng(7)
    x = (np.stack([k // (side * side), (k // side) % side, k % side], 1) + 0.5) * a
    s = w.two_atoms(5.0, box_len=side * a)
    s = s.replace(pos=x, types=(k % 3 == 0).astype(np.int32), mol=(k // 3).astype(np.int32),
                  excl_offsets=np.zeros(n + 1, np.int32))
    mass = np.where(k % 2 == 0, 15.0, 14.0)
    v0 = rng.normal(scale=3e-3, size=(n, 3))
    res = []
    for lanes in ((1, 1), (1, 1), (4, 16), (4, 16)):      # 3100 and 14000 partials
        print(f"[md] {n} atoms, lanes {lanes}", flush=True)
        rr = make_relres(s, 64)
        rr.set_launch(*lanes)
        p, v = torch.from_numpy(x).cuda(), torch.from_numpy(v0).cuda()
        rr.build_lists(p, s.box)
        rr.md_setup(mass, 1.0, 300.0, 100.0, rebuild_every=4)
        th = rr.md_run(p, v, 6, 1)
        torch.cuda.synchronize()
        res.append((p.cpu().numpy(), v.cpu().numpy(), th.cpu().numpy()))
        rr.close()
    bound = 3 * n * 2.0 ** -53
    for p, v, th in res:
        kinetic = 0.5 * float((mass[:, None] * v * v).sum()) / FTM2V
        assert abs(th[-1, 5] - kinetic) <= bound * kinetic
    for one, two in ((0, 1), (2, 3)):
        assert all(np.array_equal(a, b) for a, b in zip(res[one], res[two]))
    assert np.abs(res[0][1] - res[2][1]).max() <= 2 * bound * np.abs(res[0][1]).max()
    assert np.abs(res[0][2][:, 5] - res[2][2][:, 5]).max() <= 2 * bound * res[0][2][:, 5].max()
