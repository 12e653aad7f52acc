"""The searching kernels, which serve the bases that keep no stored terms: here
on bases that have given theirs back."""
import numpy as np
import pytest
import torch

from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from oracle import bruteforce as bf
from oracle import lanczos as olz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("index_mode", [0, 1])
@pytest.mark.parametrize("threads", [64, 192, 320, 448, 704, 960, 1024])
def test_lanczos_sums_all_waves_of_a_block(threads, index_mode):
    """Every block size that tuning takes, most of them no power of two: the
    first 10 coefficients against the oracle's, as for the other sizes."""
    from paper_1804_05028_amd import ed
    w = wl.square_4x4()
    m = bf.Model.from_workload(w)
    st, stab = bf.basis(m, w.n_up)
    v0 = vec.normal_vector(len(st), seed=7)
    ref = olz.lanczos(lambda v: bf.apply(m, st, stab, v)[0], v0, 10)
    b = ed.Basis.from_workload(w, {"block_threads": threads, "index_mode": index_mode})
    try:
        print(f"[searching] {threads} threads", flush=True)
        b.release_terms()
        r = b.lanczos(w.J, torch.as_tensor(v0).cuda(), 10)
        assert np.abs(r["alpha"] - ref["alpha"]).max() < 1e-11
        assert np.abs(r["beta"] - ref["beta"]).max() < 1e-11
    finally:
        b.close()
