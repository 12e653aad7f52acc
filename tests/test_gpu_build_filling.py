"""Basis build at every filling: the build passes over blocks of prefixes that
cannot have the sector's number of up spins.  Representatives and norms against
a plain enumeration of all configurations."""
import itertools
import math

import numpy as np
import pytest

from ed_inputs import lattice as lat
from ed_inputs import workloads as wl

pytestmark = pytest.mark.gpu


def _enumerated(perm, n_up):
    """(representatives, stabiliser sizes) of the trivial irrep, ascending: the
    few spins of one kind are placed, the others follow."""
    n = perm.shape[1]
    k = min(n_up, n - n_up)
    pos = np.array(list(itertools.combinations(range(n), k)), dtype=np.intp).reshape(math.comb(n, k), k)
    bit = np.uint64(1) << (n - 1 - perm).astype(np.uint64)   # of every site's image
    full = np.uint64((1 << n) - 1)

    def image(g):
        v = np.zeros(len(pos), np.uint64)
        for j in range(k):
            v |= bit[g][pos[:, j]]
        return v if k == n_up else v ^ full

    e = int(np.nonzero((perm == np.arange(n)).all(axis=1))[0][0])
    s = image(e)
    rep, stab = s.copy(), np.zeros(len(s), np.uint16)
    for g in range(len(perm)):
        t = image(g)
        stab += (t == s)
        rep = np.minimum(rep, t)
    own = rep == s
    order = np.argsort(s[own])
    return s[own][order], stab[own][order]


CASES = [(n, sub, k) for n, sub in ((16, 4), (20, 4), (20, 2)) for k in range(n + 1)]
CASES += [(n, sub, k) for n, sub in ((40, 5), (44, 4), (48, 6), (56, 7))
          for k in (0, 1, 3, 4, n - 4, n - 3, n)]
CASES += [(56, 8, 3), (50, 5, 4), (50, 5, 47)]


@pytest.mark.parametrize("n,sub,n_up", CASES, ids=[f"chain{n}_s{s}_n{k}" for n, s, k in CASES])
def test_build_at_every_filling(n, sub, n_up):
    from paper_1804_05028_amd import ed
    c = lat.chain(n, superlattice_period=sub)
    b = ed.Basis.from_workload(wl.Workload(f"chain{n}", c, lat.characters(c, 0), n_up, np.ones(n)))
    try:
        print(f"[build] chain{n}, {n_up} up: D={b.dim} in {b.info()['build_ms']:.2f} ms", flush=True)
        st, stab = _enumerated(np.asarray(c.perm), n_up)
        assert np.array_equal(b.states(), st)
        assert np.array_equal(b.norms(), stab)
    finally:
        b.close()
