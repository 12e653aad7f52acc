"""What a basis with stored terms keeps between calls, and what may not depend
on it: the coefficients that a captured H.v reads, and the sums of a Lanczos
call."""
import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from oracle import bruteforce as bf
from oracle import lanczos as olz

pytestmark = pytest.mark.gpu


def _square24(k=0):
    c = lat.square((6, 0), (0, 4), rotations=False, superlattice=wl.SQ_2X2)
    return wl.Workload("square24", c, lat.characters(c, k), 12, np.ones(c.n_bonds))


def _vector(b, seed=21):
    return torch.as_tensor(vec.normal_vector(b.dim, seed=seed, complex_=b.is_complex)).cuda()


@pytest.mark.parametrize("make", [wl.square_4x4, _square24], ids=["one_launch", "square24"])
@pytest.mark.parametrize("last_bit", [False, True])
def test_replay_uses_the_current_exchange(make, last_bit):
    """A captured XXZ H.v reads the handle's couplings when it is replayed
    (the Ising sum is fixed by the capture, so Jz stays).  Exchange couplings
    whose last bit differs within an orbit take another path in the eager call;
    the replay then has one value per orbit, within an eps of each bond's: a
    few eps of the row's sums."""
    from paper_1804_05028_amd import ed
    w = make()
    b = ed.Basis.from_workload(w)
    try:
        print(f"[state] {w.name}: D={b.dim}", flush=True)
        Jz = 0.4 * w.J
        x, y = _vector(b), b.empty()
        b.apply(w.J, x, out=y, Jz=Jz)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            b.apply(w.J, x, out=y, Jz=Jz)
        for f in (1.7, 0.6, 1.0):
            J = f * w.J
            if last_bit:
                J[-1] = np.nextafter(J[-1], 10.0)
            want = b.apply(J, x, Jz=Jz)
            y.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.linalg.vector_norm(y - want) <= 1e-14 * torch.linalg.vector_norm(want)
    finally:
        b.close()


def _square32(k, n_up):
    c = lat.square((4, 4), (-4, 4), rotations=False, superlattice=wl.SQ_2X2)
    return wl.Workload("square32", c, lat.characters(c, k), n_up, np.ones(c.n_bonds))


# inputs above 32 MB: real, complex and fermionic
LARGE = [("real", lambda: _square32(0, 12)), ("complex", lambda: _square32(1, 11)),
         ("fermions", lambda: wl.triangular_36_tV(n_part=13))]


def _basis(w, tuning=None):
    from paper_1804_05028_amd import ed
    return (ed.FermionBasis if hasattr(w, "t") else ed.Basis).from_workload(w, tuning)


def _lanczos(b, w, v0, steps):
    if hasattr(w, "t"):
        return b.lanczos(w.t, v0, steps, want_psi0=True, V=w.V)
    return b.lanczos(w.J, v0, steps, want_psi0=True)


def _same(r, s, n):
    return np.array_equal(r["alpha"][:n], s["alpha"][:n]) and np.array_equal(r["beta"][:n], s["beta"][:n])


@pytest.mark.parametrize("name,make", LARGE, ids=[c[0] for c in LARGE])
def test_lanczos_does_not_depend_on_the_table(name, make):
    """Stored or searched, one start vector gives one alpha and beta."""
    w = make()
    b = _basis(w)
    try:
        print(f"[state] {name}: D={b.dim}", flush=True)
        assert (b.dim + 1) * (16 if b.is_complex else 8) > 32 << 20
        v0 = _vector(b)
        r = _lanczos(b, w, v0, 5)
        b.release_terms()
        s = _lanczos(b, w, v0, 5)
        assert _same(r, s, 5)
        assert torch.equal(r["psi0"], s["psi0"])
    finally:
        b.close()


def _fermions24(k):
    c = lat.square((6, 0), (0, 4), rotations=False, superlattice=wl.SQ_2X2)
    return wl.FermionWorkload("fermions24", c, lat.characters(c, k), 12, np.ones(c.n_bonds), np.full(c.n_bonds, 0.7))


# sector, a limit in MiB that holds some of its rows (about a third to two thirds
# of its words): the call stores the first rows and searches the others
PARTIAL = [("real", lambda: _square24(0), 8), ("complex", lambda: _square24(5), 9),
           ("fermions", lambda: _fermions24(0), 8), ("fermions_complex", lambda: _fermions24(5), 9),
           ("real_large", lambda: _square32(0, 12), 500), ("complex_large", lambda: _square32(1, 11), 320),
           ("fermions_large", lambda: wl.triangular_36_tV(n_part=13), 1000)]


@pytest.mark.parametrize("name,make,mb", PARTIAL, ids=[c[0] for c in PARTIAL])
def test_lanczos_call_with_a_partial_table(name, make, mb):
    """No table (-1), one that holds the first rows only, and one of all rows:
    the same coefficients, bit for bit above 32 MB per vector, else within a few
    times sqrt(rows) eps of terms of order 10 to 20 for the first steps; H.v is
    the same in between."""
    from paper_1804_05028_amd import _lib as L
    w = make()
    out = []
    for limit in (-1, mb, 0):
        b = _basis(w, {"stored_terms_mb": limit})
        try:
            held = L.ed_basis_terms_bytes(b.handle)
            print(f"[state] {name}: D={b.dim} limit {limit} MiB, kept {held >> 20}", flush=True)
            assert (held > 0) == (limit == 0)
            if limit == 0:   # the smaller limit holds an eighth at least, and not all
                assert held / 8 < mb << 20 < held * 0.95
            x = _vector(b)
            y = b.apply(w.t, x, V=w.V) if hasattr(w, "t") else b.apply(w.J, x)
            r = _lanczos(b, w, x, 12)
            z = b.apply(w.t, x, V=w.V) if hasattr(w, "t") else b.apply(w.J, x)
            assert torch.equal(y, z) and L.ed_basis_terms_bytes(b.handle) == held
            out.append((r, y))
            large = (b.dim + 1) * (16 if b.is_complex else 8) > 32 << 20
        finally:
            b.close()
    (s, y), rest = out[0], out[1:]
    assert large == name.endswith("large")
    for r, z in rest:
        assert torch.equal(y, z) and r["n_done"] == s["n_done"] == 12
        if large:
            assert _same(r, s, 12) and torch.equal(r["psi0"], s["psi0"])
        else:
            assert np.abs(r["alpha"] - s["alpha"]).max() <= 1e-11
            assert np.abs(r["beta"] - s["beta"]).max() <= 1e-11
            # the same vector: s_j and v_j differ by what alpha and beta do
            d = torch.vdot(r["psi0"], s["psi0"]).abs().item()
            assert abs(d - 1.0) <= 1e-9


def test_table_limit_is_checked():
    from paper_1804_05028_amd import _lib as L
    with pytest.raises(L.EDError) as e:
        _basis(wl.square_4x4(), {"stored_terms_mb": -2})
    assert e.value.name == "ED_ERR_ARG"
    b = _basis(wl.square_4x4(), {"stored_terms_mb": 1})
    assert 0 < L.ed_basis_terms_bytes(b.handle) <= 1 << 20
    b.close()


def _chain(n, sub, k, n_up):
    c = lat.chain(n, superlattice_period=sub)
    return wl.Workload(f"chain{n}", c, lat.characters(c, k), n_up, np.ones(c.n_bonds))


def _open16():
    c = lat.chain(16, superlattice_period=2)
    c.perm, c.flip = c.perm[:1], c.flip[:1]
    return wl.Workload("open16", c, np.ones(1, complex), 5, np.linspace(0.5, 1.5, c.n_bonds))


# the sides of the 4096 (complex: 2048) rows up to which one launch does all steps
ROUTES = [("square16", wl.square_4x4), ("square16_k5", lambda: wl.square_4x4(momentum_index=5)),
          ("open16_4368", _open16), ("chain18_k1_2704", lambda: _chain(18, 3, 1, 9))]


@pytest.mark.parametrize("released", [False, True])
@pytest.mark.parametrize("name,make", ROUTES, ids=[c[0] for c in ROUTES])
def test_every_lanczos_route_matches_the_oracle(name, make, released):
    """One launch, two kernels a step over stored terms, and searched steps."""
    w = make()
    m = bf.Model.from_workload(w)
    st, stab = bf.basis(m, w.n_up)
    v0 = vec.normal_vector(len(st), seed=7, complex_=w.is_complex)
    ref = olz.lanczos(lambda v: bf.apply(m, st, stab, v)[0], v0, 60)
    b = _basis(w)
    try:
        if released:
            b.release_terms()
        r = b.lanczos(w.J, torch.as_tensor(v0).cuda(), 60, want_psi0=True)
        assert np.abs(r["alpha"][:10] - ref["alpha"][:10]).max() < 1e-11
        assert np.abs(r["beta"][:10] - ref["beta"][:10]).max() < 1e-11
        assert abs(r["eigenvalues"][0] - ref["eigenvalues"][0]) < 1e-10
        assert abs(torch.linalg.vector_norm(r["psi0"]).item() - 1.0) < 1e-12
    finally:
        b.close()
