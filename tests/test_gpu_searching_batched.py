"""The batched searching kernel: the tests written for it (lanes per row,
characters in LDS, in HBM and as signs, one- and two-stage search) run again
with stored terms declined."""
import pytest

from paper_1804_05028_amd import _lib as L
from tests.test_gpu_batched import (built, test_batched_apply_matches_oracle_per_sector,  # noqa: F401
                                    test_batched_lanczos_graph_replays_match_eager,
                                    test_batched_lanczos_matches_oracle, test_batched_matches_single_sector_path)
from tests.test_gpu_batched_lanes import (test_benchmark_instances_match_oracle, test_lanes_per_row_bit_identical,  # noqa: F401
                                          test_more_than_32_sectors)
from tests.test_gpu_search import test_batched_two_stage_matches_one_stage_and_oracle  # noqa: F401
from tests.test_gpu_searching import no_stored_terms  # noqa: F401

pytestmark = pytest.mark.gpu


def test_terms_are_declined(built):
    assert all(L.ed_multi_terms_bytes(mb.handle) == 0 for mb in built.values())
