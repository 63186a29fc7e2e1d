"""Bonded forces on atoms of many terms, whose force slots a wave adds up: one
term to the most an atom may have (4096), around the number that one thread
adds, several such atoms in one wave, in one block and in several, one and many
passes of slots.  Forces, energies and virial against the oracle at the bars of
the bonded forces (1e-11 relative RMS, 1e-12)."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,hubs", [(1, 3), (31, 3), (32, 3), (33, 3), (64, 10), (200, 3),
                                         (2048, 1), (2049, 2), (4090, 2)])
def test_atoms_of_many_terms(degree, hubs):
    import torch
    s = w.hexane_liquid(3, n_mol=max(120, (degree + 40) // 6 + 2), density=0.012, precision=64)
    s = s.replace(pos=s.pos + np.random.default_rng(9).normal(scale=0.05, size=s.pos.shape))
    b = dict(s.bonded)
    rng = np.random.default_rng(degree)
    bonds = [np.asarray(b["bonds"], np.int32)]
    for h in range(hubs):                       # neighbours in one wave, then apart
        hub = h if h < hubs - 1 else s.n - 1
        other = rng.choice(np.setdiff1d(np.arange(s.n), [hub]), degree, replace=False)
        bonds.append(np.stack([np.full(degree, hub), other], 1).astype(np.int32))
    b["bonds"] = np.concatenate(bonds)
    more = len(b["bonds"]) - len(b["bond_k"])
    b["bond_k"] = np.append(b["bond_k"], np.full(more, 0.7))
    b["bond_r0"] = np.append(b["bond_r0"], np.full(more, 8.0))
    s = s.replace(bonded=b)
    print(f"[bonded] {hubs} atoms of {degree} bonds, N={s.n}", flush=True)
    rr = make_relres(s, 64)
    rr.set_bonded(s.bonded)
    p = torch.from_numpy(np.ascontiguousarray(s.pos)).cuda()
    rr.build_lists(p, s.box)
    F = torch.zeros((s.n, 3), dtype=torch.float64, device="cuda")
    E, W = rr.bonded_forces(p, F)
    F2 = torch.zeros_like(F)
    rr.bonded_forces(p, F2, want_energy=False)
    torch.cuda.synchronize()
    Fb, Eb, Wb = oracle.bonded(s)
    F14, E14, W14 = oracle.pairs14(s)
    assert rel_rms(F.cpu().numpy(), Fb + F14) <= 1e-11 and rel_rms(F2.cpu().numpy(), Fb + F14) <= 1e-11
    want = np.array([Eb[0], Eb[1], Eb[2], E14[0]])
    assert np.abs(E.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    assert np.abs(W.cpu().numpy() - Wb - W14).max() <= 1e-12 * np.abs(Wb + W14).max()
    rr.close()
