"""Streamed units whose execution and idle times are taken by a workgroup each: all of the longest ones, only those beyond a line, or
none, by how many there are; against the CPU oracle."""
import numpy as np
import pytest

from paper_2311_10359_amd import traces
from parity_util import check_profile, kernels_of

pytestmark = pytest.mark.gpu
LONG = 1 << 18


@pytest.mark.parametrize("tasks,shares", [
    (3, (0.55, 0.27)),       # both units of every task in parts
    (64, (0.55, 0.27)),      # as many as there are workgroups for
    (66, (0.55, 0.27)),      # only the first of every task
    (130, (0.55, 0.27)),     # none
    (2, (0.25, 0.2503)),     # 65,536 launches and a few more
])
def test_parts(tasks, shares):
    rng = np.random.default_rng(tasks)
    kid = np.full(LONG, 2, np.uint32)
    first, second = (int(s * LONG) for s in shares)
    kid[:first], kid[first:first + second] = 0, 1
    kid[first + second:] = 2 + rng.integers(0, 300, LONG - first - second)
    kid = rng.permutation(kid)
    rec = np.zeros(LONG, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = kid * 7919, 1, 64
    ex = np.maximum(1, np.rint(rng.lognormal(8.5, 1.2, LONG))).astype(np.int64)
    gap = np.where(rng.random(LONG) < 0.3, 0, np.rint(rng.lognormal(9.6, 1.2, LONG))).astype(np.int64)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    rec["run"] = np.where(kid == 1, np.arange(LONG), 0) // 3       # the second kernel is often the last of a run
    with kernels_of() as names:
        check_profile(np.tile(rec, tasks), np.arange(tasks + 1, dtype=np.uint64) * LONG)
    assert "k_onesweep_pass" not in names, sorted(names)
