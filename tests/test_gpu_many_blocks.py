"""Many sublattices: a block's position takes more than the four bits of a 2-byte
table entry above 16 blocks, and a word of 32 tied blocks does not do above 32
(blocks of one site, with which any permutation group is stable).  Bases, H.v,
adjoint and batched H.v against the oracle."""
import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from oracle import bruteforce as bf

pytestmark = pytest.mark.gpu

# sites, blocks, up spins
SHAPES = [(16, 16, 6), (32, 16, 3), (17, 17, 8), (34, 17, 3), (36, 18, 3), (20, 20, 7), (40, 20, 3), (24, 24, 4),
          (32, 32, 3), (33, 33, 3), (40, 40, 3), (56, 56, 3)]
TUNINGS = [{}, {"table_entry_bytes": 1}, {"table_entry_bytes": 2}, {"stored_terms_mb": -1}, {"index_mode": 1}]


def _chain(n, blocks, k, n_up):
    c = lat.chain(n, superlattice_period=blocks)
    assert c.n_sublat == blocks
    return wl.Workload(f"chain{n}", c, lat.characters(c, k), n_up, np.ones(c.n_bonds))


@pytest.mark.parametrize("k", [0, 1])
@pytest.mark.parametrize("n,blocks,n_up", SHAPES, ids=[f"{n}_in_{b}" for n, b, _ in SHAPES])
def test_many_blocks(n, blocks, n_up, k):
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = _chain(n, blocks, k, n_up)
    m = bf.Model.from_workload(w)
    st, stab = bf.basis(m, n_up)
    x = vec.normal_vector(len(st), seed=5, complex_=w.is_complex)
    gy = vec.normal_vector(len(st), seed=6, complex_=w.is_complex)
    ref, kept, dropped = bf.apply(m, st, stab, x)
    ref_gx = bf.apply(m, st, stab, gy)[0]
    xd, gd = torch.as_tensor(x).cuda(), torch.as_tensor(gy).cuda()
    for tuning in TUNINGS:
        b = ed.Basis.from_workload(w, tuning)
        try:
            print(f"[blocks] {n} sites in {blocks} blocks, k={k}: D={b.dim} {tuning}", flush=True)
            assert np.array_equal(b.states(), st) and np.array_equal(b.norms(), stab)
            assert b.stats() == (len(st), kept, dropped)
            y, gx = b.apply(w.J, xd), b.empty()
            gJ = L.ed_apply_H_backward(b.handle, w.J, xd, gd, gx, True, None)
            assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
            assert np.linalg.norm(gx.cpu().numpy() - ref_gx) <= 1e-12 * np.linalg.norm(ref_gx)
            # J = 1: the bonds' sums add up to Re <gy, H x>
            assert abs(gJ.sum() - np.real(np.vdot(gy, ref))) <= 1e-12 * np.abs(gJ).sum()
            if "table_entry_bytes" not in tuning:
                assert b.info()["table_entry_bytes"] == (2 if blocks <= 16 else 4)
        finally:
            b.close()


@pytest.mark.parametrize("terms", [0, -1])
@pytest.mark.parametrize("n,blocks,n_up", [(17, 17, 8), (36, 18, 3), (40, 40, 3)], ids=["17_in_17", "36_in_18", "40_in_40"])
def test_many_blocks_batched(n, blocks, n_up, terms):
    from paper_1804_05028_amd import ed
    ws = [_chain(n, blocks, k, n_up) for k in (0, 1, 4)]
    mb = ed.MultiBasis.from_workloads(ws, {"stored_terms_mb": terms})
    try:
        rng = np.random.default_rng(3)
        x = rng.standard_normal((mb.dim, mb.K)) + 1j * rng.standard_normal((mb.dim, mb.K))
        y, masks = mb.apply(ws[0].J, torch.as_tensor(x).cuda()).cpu().numpy(), mb.masks()
        for k, w in enumerate(ws):
            m = bf.Model.from_workload(w)
            st, stab = bf.basis(m, n_up)
            sel = ((masks >> np.uint64(k)) & np.uint64(1)).astype(bool)
            assert np.array_equal(mb.states()[sel], st)
            ref = bf.apply(m, st, stab, x[sel, k])[0]
            assert np.linalg.norm(y[sel, k] - ref) <= 1e-12 * np.linalg.norm(ref)
    finally:
        mb.close()


@pytest.mark.parametrize("n,blocks,n_part", [(20, 20, 5), (34, 17, 3), (36, 36, 3)], ids=["20_in_20", "34_in_17", "36_in_36"])
def test_many_blocks_fermions(n, blocks, n_part):
    from paper_1804_05028_amd import ed
    c = lat.chain(n, superlattice_period=blocks)
    w = wl.FermionWorkload(f"ring{n}", c, lat.characters(c, 1), n_part, np.ones(n), np.full(n, 0.7))
    m = bf.FermionModel(c.n_sites, c.perm, w.chi, c.bonds, w.t, w.V)
    st, stab = bf.fbasis(m, n_part)
    x = vec.normal_vector(len(st), seed=9, complex_=True)
    ref = bf.fapply(m, st, stab, x)[0]
    for tuning in ({}, {"stored_terms_mb": -1}):
        b = ed.FermionBasis.from_workload(w, tuning)
        try:
            assert np.array_equal(b.states(), st)
            y = b.apply(w.t, torch.as_tensor(x).cuda(), V=w.V).cpu().numpy()
            assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)
        finally:
            b.close()
