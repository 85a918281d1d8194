"""Short tasks of many kernels: as many rows as fit the arrays that they are staged in, one array's worth, one row more or less;
against the CPU oracle, and whether the sort was needed."""
import numpy as np
import pytest

from paper_2311_10359_amd import traces
from parity_util import check_profile, kernels_of

pytestmark = pytest.mark.gpu


def task(rng, launches, ids):
    kid = np.concatenate([np.arange(ids), rng.integers(0, ids, launches - ids)]).astype(np.uint32)
    rec = np.zeros(launches, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = rng.permutation(kid) * 7919, 1, 64
    ex, gap = rng.integers(1, 1 << 20, launches), rng.integers(0, 1 << 31, launches)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    rec["run"] = np.arange(launches) // 7
    return rec


@pytest.mark.parametrize("launches", [8, 9, 15, 16, 17, 63, 100, 341, 342, 700, 5000, 9000])
def test_rows_at_the_edges_of_their_room(launches):
    rng = np.random.default_rng(launches)
    each, most = launches // 8, 512 if launches > 8192 else 256
    counts = sorted({min(c, launches, most) for c in (1, each - 1, each, each + 1, 2 * each, 5 * each + 1, 6 * each - 1, 6 * each, 6 * each + 1, launches)
                     if c > 0})
    for ids in counts:
        print(f"{launches} launches, {ids} kernels", flush=True)
        recs = [task(rng, 20, 3), task(rng, launches, ids), task(rng, launches, 1), task(rng, 300, 40)]   # (beside others, before and behind)
        off = np.concatenate([[0], np.cumsum([r.size for r in recs])]).astype(np.uint64)
        with kernels_of() as names:
            check_profile(np.concatenate(recs), off)
        assert ("k_leaf_sort" in names) == (ids > 6 * each), sorted(names)
