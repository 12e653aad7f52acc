"""What a basis with stored terms keeps between calls: the coefficients that a
captured H.v reads."""
import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl

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
