"""Profiles of so many tasks that their row offsets take several rounds of one launch, or three launches; against the CPU oracle."""
import numpy as np
import pytest

from paper_2311_10359_amd import traces
from parity_util import check_profile, kernels_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tasks", [8191, 8192, 41003, 262143, 262144, 300001])   # (one entry more than tasks; 262,144 in one launch)
def test_row_offsets_of_profiles(n_tasks):
    rng = np.random.default_rng(n_tasks)
    lens = rng.choice([0, 8, 9, 17], n_tasks)            # (from 8 launches on a task's rows are staged, and nothing is left to the sort)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    n = int(off[-1])
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = rng.integers(0, 3, n) * 7919, 1, 64
    ex, gap = rng.integers(1, 9000, n), rng.integers(0, 40000, n)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    with kernels_of() as names:
        check_profile(rec, off)
    assert "k_leaf_sort" not in names, sorted(names)
