"""Stored terms (one word per off-diagonal term, searched once per basis)
against the searching kernels on the same basis: H.v and gx must agree bit for
bit, since both sum a row's terms in bond order by the same operations.  The
per-bond sums and the Lanczos coefficients add the rows in another order; their
bound is a few times sqrt(rows) eps of the sum's terms, far below 1e-12.

The cases take every width of table entry, one and several chunks, one- and
two-stage search, real and complex sectors, fermions, couplings that differ
between bond orbits, sectors of less than a slice of 64 rows, of exactly one,
and on both sides of the 4096 (complex: 2048) rows up to which an H.v keeps its
input in LDS, the counted (not fixed-stride) layout, and the refusals: the
Limits index, too many classes, and couplings that differ in their last bit
within an orbit."""
import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from tests.test_gpu_adjoint_fused import CASES as SPIN_CASES
from tests.test_gpu_fermions import CASES as FERMI_CASES, IDS as FERMI_IDS
from tests.test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu


def _chain(n, sub, k, n_up, **kw):
    c = lat.chain(n, superlattice_period=sub, **kw)
    return wl.Workload(f"chain{n}", c, lat.characters(c, k), n_up, np.ones(c.n_bonds))


def _trivial_group(n, n_up, sub=1):
    """No symmetry but the identity: every bond an orbit of its own."""
    c = lat.chain(n, superlattice_period=sub)
    c.perm, c.flip = c.perm[:1], c.flip[:1]
    return wl.Workload("open", c, np.ones(1, complex), n_up, np.linspace(0.5, 1.5, c.n_bonds))


def _square24(k):
    c = lat.square((6, 0), (0, 4), rotations=False, superlattice=wl.SQ_2X2)
    o = lat.bond_orbits(c)
    J = np.linspace(0.7, 1.3, o.max() + 1)[o]
    return wl.Workload("square24", c, lat.characters(c, k), 12, J)


EDGES = [
    ("one_row", lambda: _chain(4, 2, 2, 2), None),
    ("chain8_1up", lambda: _chain(8, 2, 0, 1), None),
    ("chain14_k3", lambda: _chain(14, 7, 3, 5), None),
    ("rows_64", lambda: _trivial_group(64 // 8, 1), None),
    ("no_symmetry_924", lambda: _trivial_group(12, 6), None),
    ("no_symmetry_3432", lambda: _trivial_group(14, 7, 2), None),
    ("no_symmetry_4368", lambda: _trivial_group(16, 5, 2), None),    # above the LDS bound, real
    ("chain18_k1", lambda: _chain(18, 3, 1, 9), None),               # complex, 2704 rows
    ("chain16_k1", lambda: _chain(16, 4, 1, 8), None),               # complex, 800 rows
    ("square24_k0", lambda: _square24(0), None),                     # 1.1e5 rows, counted layout
    ("square24_k5", lambda: _square24(5), None),
]
CASES = EDGES + [c for c in SPIN_CASES if c[0] != "square32_disorder"] + [(n, (lambda w=w: w), None) for n, w in SMALL]


def _square32(k, n_up):
    c = lat.square((4, 4), (-4, 4), rotations=False, superlattice=wl.SQ_2X2)
    return wl.Workload("square32", c, lat.characters(c, k), n_up, np.ones(c.n_bonds))


def _vectors(b):
    return [torch.as_tensor(vec.normal_vector(b.dim, seed=s, complex_=b.is_complex)).cuda() for s in (21, 22)]


@pytest.mark.parametrize("name,make,tuning", CASES, ids=[c[0] for c in CASES])
def test_stored_terms_equal_search(name, make, tuning):
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = make()
    b = ed.Basis.from_workload(w, tuning)
    try:
        print(f"[terms] {name}: D={b.dim}", flush=True)
        assert L.ed_basis_terms_bytes(b.handle) > 0 or b.dim == 0
        o = lat.bond_orbits(w.cluster)
        J = lat.orbit_mean(np.asarray(w.J, np.float64), o)
        Jz = J * 0.37
        x, gy = _vectors(b)
        steps = max(1, min(12, b.dim // 3))

        def all_of():
            gx = b.empty()
            gJ = L.ed_apply_H_backward(b.handle, J, x, gy, gx, True, None)
            alone = L.ed_apply_H_backward(b.handle, J, x, gy, None, True, None)
            assert np.array_equal(gJ, alone)
            r = b.lanczos(J, x, steps, want_psi0=True, Jz=Jz)
            return b.apply(J, x), b.apply(J, x, Jz=Jz), gx, gJ, r

        a = all_of()
        # couplings with one value off by a bit within an orbit: searched bond by bond
        big = int(np.argmax(np.bincount(o)))
        if np.bincount(o)[big] > 1:
            J2 = J.copy()
            k = np.nonzero(o == big)[0][-1]
            J2[k] = np.nextafter(J2[k], 2.0)
            y2 = b.apply(J2, x)
        b.release_terms()
        assert L.ed_basis_terms_bytes(b.handle) == 0
        s = all_of()
        torch.cuda.synchronize()
        assert torch.equal(a[0], s[0]) and torch.equal(a[1], s[1]) and torch.equal(a[2], s[2])
        if np.bincount(o)[big] > 1:
            assert torch.equal(y2, b.apply(J2, x))
        scale = max(1.0, np.abs(s[3]).max())
        assert np.abs(a[3] - s[3]).max() <= 1e-12 * scale
        assert a[4]["n_done"] == s[4]["n_done"]
        assert np.abs(a[4]["alpha"] - s[4]["alpha"]).max() <= 1e-11
        assert np.abs(a[4]["beta"] - s[4]["beta"]).max() <= 1e-11
    finally:
        b.close()


@pytest.mark.parametrize("w,tune", FERMI_CASES, ids=FERMI_IDS)
def test_stored_terms_equal_search_fermions(w, tune):
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    b = ed.FermionBasis.from_workload(w, tune)
    try:
        print(f"[terms] {w.name}: D={b.dim}", flush=True)
        assert L.ed_basis_terms_bytes(b.handle) > 0 or b.dim == 0
        if b.dim == 0:
            return
        x, _ = _vectors(b)
        a = b.apply(w.t, x, V=w.V), b.apply(w.t, x)
        b.release_terms()
        assert torch.equal(a[0], b.apply(w.t, x, V=w.V)) and torch.equal(a[1], b.apply(w.t, x))
    finally:
        b.close()


# inputs on both sides of the 32 MB above which slices come from a counter
COUNTED = [("square32_n11", 0, 11, False), ("square32_n12", 0, 12, True), ("square32_k1_n10", 1, 10, False),
           ("square32_k1_n11", 1, 11, True)]


@pytest.mark.parametrize("name,k,n_up,counted", COUNTED, ids=[c[0] for c in COUNTED])
def test_slice_counter(name, k, n_up, counted):
    """Repeated H.v and Lanczos calls with slices taken from a counter give the
    same bits each time, and those of the searching kernels."""
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = _square32(k, n_up)
    b = ed.Basis.from_workload(w)
    try:
        print(f"[terms] {name}: D={b.dim}", flush=True)
        assert (b.dim * (16 if b.is_complex else 8) > 32 << 20) == counted
        x, gy = _vectors(b)
        y = b.apply(w.J, x)
        z = b.apply(w.J, gy)
        assert torch.equal(y, b.apply(w.J, x)) and torch.equal(z, b.apply(w.J, gy))
        r = b.lanczos(w.J, x, 5)
        r2 = b.lanczos(w.J, x, 5)
        assert np.array_equal(r["alpha"], r2["alpha"]) and np.array_equal(r["beta"], r2["beta"])
        gx = b.empty()
        L.ed_apply_H_backward(b.handle, w.J, x, gy, gx, True, None)
        assert torch.equal(gx, z)
        b.release_terms()
        assert torch.equal(y, b.apply(w.J, x)) and torch.equal(z, b.apply(w.J, gy))
        s = b.lanczos(w.J, x, 5)
        assert np.abs(r["alpha"] - s["alpha"]).max() <= 1e-11 and np.abs(r["beta"] - s["beta"]).max() <= 1e-11
    finally:
        b.close()


def test_terms_of_a_lanczos_call():
    """A sector whose terms are too many to keep: a Lanczos call of 16 steps
    stores all of them, or (here, where little memory is free) those of the
    first rows, and gives the memory back.  The sums add the rows in another
    order than the searching call: a few times sqrt(rows) eps of terms of order
    20, below 1e-9.  A coupling that differs by a bit within its orbit is
    searched, and so is every call after the release."""
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = wl.square_40_j1j2(n_sub=4)
    b = ed.Basis.from_workload(w)
    try:
        print(f"[terms] square40: D={b.dim}", flush=True)
        assert L.ed_basis_terms_bytes(b.handle) == 0
        states = b.states_device()
        x = vec.hashed_amplitudes_torch(states, salt=1, complex_=False)
        del states
        torch.cuda.empty_cache()
        few = b.lanczos(w.J, x, 4)                    # searched; the vectors stay with the basis
        y = b.apply(w.J, x)
        free, held = torch.cuda.mem_get_info()[0], b.info()["device_bytes"]
        most = b.lanczos(w.J, x, 16)
        fill = torch.empty(torch.cuda.mem_get_info()[0] - (80 << 30), dtype=torch.uint8, device="cuda")
        some = b.lanczos(w.J, x, 8, want_psi0=True)   # 16 steps in two passes
        psi0 = some["psi0"]
        hp = b.apply(w.J, psi0)
        del fill
        J2 = w.J.copy()
        J2[0] = np.nextafter(J2[0], 2.0)
        other = b.lanczos(J2, x, 16)
        assert torch.equal(y, b.apply(w.J, x))
        torch.cuda.empty_cache()
        assert L.ed_basis_terms_bytes(b.handle) == 0 and b.info()["device_bytes"] == held
        b.release_terms()
        s = b.lanczos(w.J, x, 16)
        for r, n in ((few, 4), (most, 16), (some, 8), (other, 16)):
            assert r["n_done"] == n
            assert np.abs(r["alpha"][:n] - s["alpha"][:n]).max() <= 1e-9
            assert np.abs(r["beta"][:n - 1] - s["beta"][:n - 1]).max() <= 1e-9
        assert abs(float(torch.dot(psi0, hp)) - some["eigenvalues"][0]) <= 1e-9
        assert torch.cuda.mem_get_info()[0] >= free - 2 * x.numel() * 8 - (1 << 30)
    finally:
        b.close()


def _square20(k, n_up):
    c = lat.square((4, 2), (-2, 4), j2=True, rotations=False, superlattice=wl.SQ_2X2)
    return wl.Workload("square20", c, lat.characters(c, k), n_up, wl.couplings_by_kind(c.bond_kind, [1.0, 0.5]))


def _identity16(n_up):
    """32 bond orbits of the 4x4 square: 33 classes, 6 bits."""
    c = lat.square((4, 0), (0, 4), rotations=False, superlattice=wl.SQ_2X2)
    c.perm, c.flip = c.perm[:1], c.flip[:1]
    return wl.Workload("square16", c, np.ones(1, complex), n_up, np.linspace(0.5, 1.5, c.n_bonds))


# words of the one-launch Lanczos: 16 bits in LDS for all slices, for some
# (31 slices of about 12 groups), or for none (class and row take 17 bits)
ONE_LAUNCH = [("all", lambda: _identity16(3), 24), ("some", lambda: _square20(0, 6), 24), ("none", lambda: _identity16(4), 24),
              ("complex_all", lambda: _chain(20, 4, 1, 6), 24), ("complex_none", lambda: _square20(1, 6), 24),
              ("more_steps_than_threads", lambda: _square20(0, 6), 1100)]


@pytest.mark.parametrize("name,make,steps", ONE_LAUNCH, ids=[c[0] for c in ONE_LAUNCH])
def test_lanczos_in_one_launch(name, make, steps):
    """Against the steps of the searching kernels: the first 12 coefficients
    differ by a few times sqrt(rows) eps of terms of order 10 each step, the
    extremal Ritz values stay with the sector's (converged after 1100 steps)."""
    from paper_1804_05028_amd import ed
    w = make()
    b = ed.Basis.from_workload(w)
    try:
        print(f"[terms] {name}: D={b.dim}", flush=True)
        assert b.dim <= (2048 if b.is_complex else 4096)
        x, _ = _vectors(b)
        r, again = b.lanczos(w.J, x, steps, want_psi0=True), b.lanczos(w.J, x, steps)
        assert np.array_equal(r["alpha"], again["alpha"]) and np.array_equal(r["beta"], again["beta"])
        b.release_terms()
        s = b.lanczos(w.J, x, steps)
        assert r["n_done"] == s["n_done"] == steps
        assert np.abs(r["alpha"][:12] - s["alpha"][:12]).max() <= 1e-11
        assert np.abs(r["beta"][:12] - s["beta"][:12]).max() <= 1e-11
        if steps > 1000:
            for k in (0, -1):
                assert abs(r["eigenvalues"][k] - s["eigenvalues"][k]) <= 1e-10
            assert torch.linalg.vector_norm(b.apply(w.J, r["psi0"]) - s["eigenvalues"][0] * r["psi0"]) <= 1e-7
    finally:
        b.close()


def test_refusals_and_release():
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    w = wl.square_4x4()
    b = ed.Basis.from_workload(w, {"index_mode": 1})
    assert L.ed_basis_terms_bytes(b.handle) == 0
    b.release_terms()
    b.close()
    b = ed.Basis.from_workload(w)
    held, before = L.ed_basis_terms_bytes(b.handle), b.info()["device_bytes"]
    b.release_terms()
    assert b.info()["device_bytes"] == before - held
    b.release_terms()
    b.close()


def test_captured_call_replays():
    """An H.v captured in a graph replays with new inputs and the eager result."""
    from paper_1804_05028_amd import ed
    for w in (wl.square_4x4(), _square24(0)):
        b = ed.Basis.from_workload(w)
        x, gy = _vectors(b)
        buf, y = x.clone(), b.empty()
        b.apply(w.J, buf, out=y)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            b.apply(w.J, buf, out=y)
        for v in (gy, x, gy):
            buf.copy_(v)
            g.replay()
            torch.cuda.synchronize()
            got = y.clone()
            assert torch.equal(got, b.apply(w.J, v))
        b.close()


def _multi_cases():
    from tests.test_gpu_batched import CASES as B
    from tests.test_gpu_batched_lanes import BENCH_INSTANCES
    out = [(n, ws, None) for n, ws in B]
    for n, make, tune, *_ in BENCH_INSTANCES:
        out += [(f"{n}_{lanes}", make(), dict(tune, table_entry_bytes=2, search_mode=2, lanes_per_row=lanes)) for lanes in (1, 2, 4)]
    c = lat.square((6, 0), (0, 4), rotations=False, superlattice=wl.SQ_2X2)
    J = np.linspace(0.7, 1.3, lat.bond_orbits(c).max() + 1)[lat.bond_orbits(c)]
    for K in (1, 2, 3, 5, 17, 24):   # every number of lanes per row up to 32, full and not
        out.append((f"square24_K{K}", [wl.Workload("sq24", c, lat.characters(c, k), 10, J) for k in range(K)], None))
    c = lat.chain(36, superlattice_period=9)   # 64 lanes per row
    out.append(("chain36_K33", [wl.Workload("c36", c, lat.characters(c, k), 3, np.ones(36)) for k in range(33)], None))
    return out


MULTI = _multi_cases()


@pytest.mark.parametrize("name,ws,tune", MULTI, ids=[m[0] for m in MULTI])
def test_batched_stored_terms_equal_search(name, ws, tune):
    """Batched H.v and Lanczos from stored terms against the searching kernel
    on the same basis, with values that are not finite outside the sectors.
    Both round each term a few times: a few times the terms' eps, below 1e-13
    of the norm."""
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    mb = ed.MultiBasis.from_workloads(ws, tune)
    try:
        print(f"[terms] {name}: D={mb.dim} K={mb.K}", flush=True)
        assert L.ed_multi_terms_bytes(mb.handle) > 0
        rng = np.random.default_rng(5)
        x = rng.standard_normal((mb.dim, mb.K)) + 1j * rng.standard_normal((mb.dim, mb.K))
        out = ((mb.masks()[:, None] >> np.arange(mb.K, dtype=np.uint64)) & np.uint64(1)) == 0
        x[out] = np.nan
        x = torch.as_tensor(x).cuda()
        v0 = torch.where(torch.isnan(x.real), torch.zeros_like(x), x)
        y, r = mb.apply(ws[0].J, x), mb.lanczos(ws[0].J, v0, 4)
        again = mb.apply(ws[0].J, x)
        eager = mb.lanczos(ws[0].J, v0, 4, use_graph=False)
        assert torch.equal(y, again)
        assert np.array_equal(r["alpha"], eager["alpha"]) and np.array_equal(r["beta"], eager["beta"])
        mb.release_terms()
        assert L.ed_multi_terms_bytes(mb.handle) == 0
        z, s = mb.apply(ws[0].J, x), mb.lanczos(ws[0].J, v0, 4)
        assert not torch.isnan(y.real).any() and (y[torch.as_tensor(out).cuda()] == 0).all()
        assert torch.linalg.vector_norm(y - z) <= 1e-13 * torch.linalg.vector_norm(z)
        assert np.array_equal(r["n_done"], s["n_done"])
        for k in range(mb.K):
            n = int(r["n_done"][k])
            if np.all(s["beta"][k, :max(n - 1, 0)] > 1e-6):   # no breakdown on the way
                assert np.abs(r["alpha"][k, :n] - s["alpha"][k, :n]).max(initial=0.0) <= 1e-11
    finally:
        mb.close()
