"""The searching kernels, which serve the bases that keep no stored terms.  The
tests imported here were written for them (index and table variants, every wave
of a block, one- and two-stage search, fermionic signs, the fused adjoint) and
run again with stored terms declined; in their own modules the same bases store
their terms."""
import numpy as np
import pytest
import torch

from ed_inputs import lattice as lat
from ed_inputs import vectors as vec
from ed_inputs import workloads as wl
from oracle import bruteforce as bf
from oracle import lanczos as olz
from tests.test_gpu_adjoint import test_backward_matches_oracle  # noqa: F401
from tests.test_gpu_adjoint_fused import test_fused_adjoint_equals_separate_products  # noqa: F401
from tests.test_gpu_edges import test_edge_sizes_match_oracle  # noqa: F401
from tests.test_gpu_fermions import test_fermion_basis_hv_and_lanczos  # noqa: F401
from tests.test_gpu_parity import (built, test_apply_parity, test_every_wave_of_a_block_complex_and_fermionic,  # noqa: F401
                                   test_every_wave_of_a_block_with_one_byte_single_chunk_tables,
                                   test_index_and_table_variants, test_lanczos_breakdown_small_sector,
                                   test_lanczos_eigenvalues, test_lanczos_ground_state_vector,
                                   test_lanczos_near_breakdown_matches_oracle_step_count)
from tests.test_gpu_search import (test_two_stage_lanczos_matches_oracle,  # noqa: F401
                                   test_two_stage_matches_one_stage_and_oracle)
from tests.test_gpu_xxz import test_xxz_apply_and_lanczos_match_oracle  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def no_stored_terms():
    from paper_1804_05028_amd import _lib as L
    tuning = L._tuning

    def declined(t):
        out = tuning(t or {})
        out.stored_terms_mb = -1
        return out

    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(L, "_tuning", declined)
        yield


def test_terms_are_declined():
    from paper_1804_05028_amd import _lib as L
    from paper_1804_05028_amd import ed
    b = ed.Basis.from_workload(wl.square_4x4())
    assert L.ed_basis_terms_bytes(b.handle) == 0
    b.close()


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
        r = b.lanczos(w.J, torch.as_tensor(v0).cuda(), 10)
        assert np.abs(r["alpha"] - ref["alpha"]).max() < 1e-11
        assert np.abs(r["beta"] - ref["beta"]).max() < 1e-11
    finally:
        b.close()
