"""The tuner on bases that store their terms: the fields it varies steer the
searching kernels, so that it must not choose among them by noise."""
import numpy as np
import pytest

from ed_inputs import lattice as lat
from ed_inputs import workloads as wl

pytestmark = pytest.mark.gpu


def test_stored_terms_are_timed_once_per_decomposition():
    from paper_1804_05028_amd import autotune as at
    make = lambda ns: wl.square_20_j1j2(n_sub=ns)
    best, results = at.autotune(make, [4, 5, 10], reps=2)
    assert [r["n_sub"] for r in results if "hv_ms" in r] == [4, 5, 10]
    assert best["tuning"] == {}
    # declined, every candidate runs a kernel of its own
    off = [{"stored_terms_mb": -1}, {"stored_terms_mb": -1, "block_threads": 256}, {"index_mode": 1}]
    best, results = at.autotune(make, [4], candidates=lambda bits: [{}] + off, reps=2)
    assert [r["tuning"] for r in results if "hv_ms" in r] == [{}] + off


def test_batched_schedule_times_one_lane_count_for_stored_terms():
    from paper_1804_05028_amd import autotune as at
    c = wl.square_4x4().cluster
    ws = [wl.Workload(f"sq16_k{k}", c, lat.characters(c, k), 8, np.ones(c.n_bonds)) for k in range(16)]
    tuned = at.autotune_batched(ws, batches=(4, 16), reps=2)
    assert [(t["K"], t["lanes_per_row"]) for t in tuned["trials"]] == [(4, 1), (16, 1)]
