"""Stored terms at the limits of their layout: more than 64, 128 and 192 bonds
(words of the bond mask, and the adjoint's sums per bond in registers up to 128
and in lanes above), real and complex, one slice and several blocks of rows, and
a sector with more classes than a table can have.  H.v, gx and gJ against the
oracle; against the searching kernels y and gx agree bit for bit."""
import itertools

import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from oracle import bruteforce as bf
from tests.test_gpu_adjoint import _oracle_per_bond

pytestmark = pytest.mark.gpu


def _rings(n, cycles, ks, n_up):
    """All pairs of n sites in two blocks; the group rotates the given rings of
    sites independently, ring c with character exp(2 pi i k_c j / length)."""
    c = lat.chain(n)
    c.n_sublat = 2
    perms, chi = [], []
    for js in itertools.product(*[range(len(s)) for s in cycles]):
        p = np.arange(n)
        phase = 0.0
        for sites, j, k in zip(cycles, js, ks):
            p[sites] = np.roll(sites, -j)
            phase += k * j / len(sites)
        perms.append(p)
        chi.append(np.exp(2j * np.pi * phase))
    c.perm = np.array(perms, dtype=np.int32)
    c.flip = np.zeros(len(perms), np.uint8)
    c.bonds = np.array(list(itertools.combinations(range(n), 2)), dtype=np.int32)
    o = lat.bond_orbits(c)
    J = np.random.default_rng(n).uniform(0.5, 1.5, o.max() + 1)[o]
    return wl.Workload(f"rings{n}", c, np.array(chi), n_up, J)


R16 = [np.arange(0, 3), np.arange(3, 8), np.arange(8, 15)]   # 105 elements, 12 orbits of 120 bonds
R20 = [np.arange(0, 5), np.arange(10, 17)]                   # 35 elements, 50 orbits of 190 bonds
R22 = [np.arange(0, 5), np.arange(11, 18)]                   # 35 elements, 231 bonds
CASES = [
    ("120_complex", lambda: _rings(16, R16, (0, 0, 1), 8), True),
    ("120_complex_blocks", lambda: _rings(16, R16[2:], (1,), 8), True),
    ("120_too_many_classes", lambda: _rings(16, R16, (1, 1, 1), 8), False),
    ("190_real", lambda: _rings(20, R20, (0, 0), 4), True),
    ("190_complex", lambda: _rings(20, R20, (0, 1), 4), True),
    ("190_too_many_classes", lambda: _rings(20, R20, (1, 1), 4), False),
    ("231_real", lambda: _rings(22, R22, (0, 0), 7), True),
    ("231_complex", lambda: _rings(22, R22, (1, 0), 7), True),
]


@pytest.mark.parametrize("name,make,stored", CASES, ids=[c[0] for c in CASES])
def test_many_bonds_and_classes(name, make, stored):
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = make()
    m = bf.Model.from_workload(w)
    st, stab = bf.basis(m, w.n_up)
    x = vec.normal_vector(len(st), seed=5, complex_=w.is_complex)
    gy = vec.normal_vector(len(st), seed=6, complex_=w.is_complex)
    xd, gd = torch.as_tensor(x).cuda(), torch.as_tensor(gy).cuda()
    b = ed.Basis.from_workload(w)
    try:
        print(f"[limits] {name}: D={b.dim}, {b.n_bonds} bonds, complex {b.is_complex}", flush=True)
        assert b.is_complex == w.is_complex and np.array_equal(b.states(), st)
        assert (L.ed_basis_terms_bytes(b.handle) > 0) == stored
        ref, kept, dropped = bf.apply(m, st, stab, x)
        ref_gx = bf.apply(m, st, stab, gy)[0]
        ref_gJ = _oracle_per_bond(w, st, stab, x, gy)
        assert b.stats() == (len(st), kept, dropped)
        got = []
        for _ in range(2 if stored else 1):
            y = b.apply(w.J, xd)
            gx = b.empty()
            gJ = L.ed_apply_H_backward(b.handle, w.J, xd, gd, gx, True, None)
            alone = L.ed_apply_H_backward(b.handle, w.J, xd, gd, None, True, None)
            noalloc = L.ed_apply_H_backward_noalloc(b.handle, w.J, xd, gd, None, True, None)
            assert np.array_equal(gJ, alone) and np.abs(noalloc - gJ).max() <= 1e-12 * np.abs(gJ).max()
            assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
            assert np.linalg.norm(gx.cpu().numpy() - ref_gx) <= 1e-12 * np.linalg.norm(ref_gx)
            assert np.abs(gJ - ref_gJ).max() <= 1e-12 * max(1.0, np.abs(ref_gJ).max())
            r = b.lanczos(w.J, xd, 8)
            got.append((y, gx, r))
            b.release_terms()
        if stored:
            (y, gx, r), (z, gz, s) = got
            assert torch.equal(y, z) and torch.equal(gx, gz)
            # sums of terms of order 100
            assert np.abs(r["alpha"] - s["alpha"]).max() <= 1e-10
            assert np.abs(r["beta"] - s["beta"]).max() <= 1e-10
    finally:
        b.close()
