"""The bonded kernel's blocks of atoms: molecules that end inside a block,
chains and random terms that straddle blocks (a term is then evaluated by
each block that owns one of its atoms, its energy and virial counted once),
atoms with more terms than a pass has force slots, and block sizes from the
smallest to the largest.  Bars as for the bonded forces elsewhere: FP64 on
both sides, 1e-11 relative RMS for forces, 1e-12 for energies and virial."""
import numpy as np
import pytest

import oracle
import workloads as w
from _util import make_relres, rel_rms

pytestmark = pytest.mark.gpu


def _system(n, seed, bonds, angles, dihedrals, pairs):
    rng = np.random.default_rng(seed)
    s = w.two_atoms(5.0, box_len=60.0)
    i32 = lambda a, k: np.asarray(a, np.int32).reshape(-1, k)      # noqa: E731
    b, a, d, p = i32(bonds, 2), i32(angles, 3), i32(dihedrals, 4), i32(pairs, 2)
    bonded = dict(bonds=b, bond_k=rng.uniform(1, 3, len(b)), bond_r0=rng.uniform(1, 2, len(b)),
                  angles=a, angle_k=rng.uniform(1, 3, len(a)), angle_t0=rng.uniform(1, 2, len(a)),
                  dihedrals=d, dih_k=rng.uniform(1, 3, len(d)),
                  dih_n=rng.integers(0, 5, len(d)).astype(np.int32), dih_d=rng.uniform(0, 3, len(d)),
                  pairs14=p, scale14=0.5, masses=np.full(n, 14.0))
    return s.replace(pos=rng.uniform(0.0, 60.0, size=(n, 3)), types=rng.integers(0, 2, n).astype(np.int32),
                     mol=np.arange(n, dtype=np.int32), excl_offsets=np.zeros(n + 1, np.int32),
                     bonded=bonded)


def _check(s, precision):
    import torch
    print(f"[bonded] N={s.n} terms={[len(s.bonded[k]) for k in ('bonds', 'angles', 'dihedrals', 'pairs14')]} "
          f"precision={precision}", flush=True)
    rr = make_relres(s, precision)
    rr.set_bonded(s.bonded)
    p = torch.from_numpy(np.ascontiguousarray(s.pos)).cuda()
    rr.build_lists(p, s.box)
    F = torch.zeros((s.n, 3), dtype=torch.float64 if precision == 64 else torch.float32, device="cuda")
    E, W = rr.bonded_forces(p, F)
    G = torch.zeros_like(F)
    rr.bonded_forces(p, G, want_energy=False)       # the launch without sums
    torch.cuda.synchronize()
    Fb, Eb, Wb = oracle.bonded(s)
    F14, E14, W14 = oracle.pairs14(s)
    assert rel_rms(F.double().cpu().numpy(), Fb + F14) <= (1e-11 if precision == 64 else 1e-5)
    assert torch.equal(F, G)
    want = np.array([Eb[0], Eb[1], Eb[2], E14[0]])
    np.testing.assert_allclose(E.cpu().numpy(), want, rtol=1e-12, atol=1e-12 * np.abs(want).max())
    Wr = Wb + W14
    assert np.abs(W.cpu().numpy() - Wr).max() <= 1e-12 * np.abs(Wr).max()
    rr.close()


def _chain(n, start=0):
    return [[[start + i + d for d in range(k)] for i in range(n - k + 1)] for k in (2, 3, 4)]


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [2, 17, 700])
def test_one_chain_straddles_blocks(n, precision):
    b, a, d = _chain(n)
    _check(_system(n, n, b, a, d, [[q[0], q[3]] for q in d]), precision)


def test_random_terms_cross_blocks():
    rng = np.random.default_rng(8)
    n = 900
    pick = lambda k, m: [rng.choice(n, k, replace=False).tolist() for _ in range(m)]    # noqa: E731
    _check(_system(n, 8, pick(2, 500), pick(3, 400), pick(4, 300), pick(2, 350)), 64)


def test_atom_with_more_terms_than_a_pass():
    """One atom in 3000 bonds and 300 angles (two passes of force slots), its
    neighbours in one each."""
    n = 3001
    bonds = [[0, j] for j in range(1, n)]
    angles = [[j, 0, j + 1] for j in range(1, 600, 2)]
    _check(_system(n, 9, bonds, angles, [], []), 64)


def test_largest_blocks_of_short_molecules():
    """30000 atoms (blocks of 96 and more, ended between molecules of 7) and a
    tail without terms."""
    n, m = 30000, 7
    b, a, d = [], [], []
    for k in range(0, n - 400, m):
        cb, ca, cd = _chain(m, k)
        b, a, d = b + cb, a + ca, d + cd
    _check(_system(n, 10, b, a, d, []), 64)
