"""Units of long tasks: IDs with as many launches as a group of lanes, a wave or a share of the workgroup takes and one more or
less, beside others that fill the unit, with values that crowd a histogram's bins; every output against the CPU oracle."""
import numpy as np
import pytest

from paper_2311_10359_amd import traces
from parity_util import check_profile, kernels_of, unit_sizes

pytestmark = pytest.mark.gpu
EDGES = [1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025]


def values(rng, kind, kid, n):
    if kind == "equal":
        return 1000 + kid % 7
    if kind == "narrow":                        # fewer values than bins, far from 0
        return 100_000_000 + rng.integers(0, 200, n)
    if kind == "two":                           # most samples at two values, and one at each end of 32 bits per ID
        v = np.where(rng.random(n) < 0.6, 4097, 70_000)
        v[np.unique(kid, return_index=True)[1]] = (1 << 32) - 2
        v[n - 1 - np.unique(kid[::-1], return_index=True)[1]] = 0
        return v
    if kind == "powers":                        # around powers of two, where a float's steps change
        return np.minimum((np.int64(1) << rng.integers(0, 32, n)) + rng.integers(-3, 4, n), (1 << 32) - 2).clip(0)
    if kind == "clustered":                     # thousands of values within one bin of a wide range
        return np.where(rng.random(n) < 0.98, 1_000_000 + rng.integers(0, 300, n), rng.integers(1, 4_000_000_000, n))
    return np.maximum(1, np.rint(rng.lognormal(9 + kid % 5, 0.3 + 0.4 * (kid % 4), n))).astype(np.int64)


def task(rng, counts, kind, first):
    kid = rng.permutation(np.repeat(first + np.arange(len(counts)), counts))
    rec = np.zeros(kid.size, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = kid * 7919, 1, 64
    ex, gap = values(rng, kind, kid, kid.size), values(rng, kind, kid, kid.size)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    # runs of one or two launches in a part of the trace: some IDs have no idle time at all, others few
    rec["run"] = np.where(kid % 11 == 3, np.arange(kid.size), np.arange(kid.size) // 5000)
    return rec


@pytest.mark.parametrize("kind", ["equal", "narrow", "two", "powers", "clustered", "lognormal"])
def test_ids_at_the_edges_of_groups_waves_and_shares(kind):
    rng = np.random.default_rng(len(kind))
    counts = [
        EDGES + [1500] * 8,                                  # just long enough to be cut into units
        EDGES * 4 + [12000, 8193, 8192, 4097, 4096, 3000],   # ... with IDs that fill a unit of each shape
        [7000, 700] + [300] * 30 + [8000] * 14,              # 131,073 launches and more: the larger units
        [20] * 2500,                                         # many IDs of few launches
    ]
    counts[2].append(max(1, 131073 - sum(counts[2])))
    recs = [task(rng, c, kind, 10_000 * i) for i, c in enumerate(counts)]
    off = np.concatenate([[0], np.cumsum([r.size for r in recs])]).astype(np.uint64)
    with kernels_of() as names:
        _, _, (ids, _, _) = check_profile(np.concatenate(recs), off)
    assert "k_onesweep_pass" not in names, sorted(names)
    sizes = unit_sizes(ids, off)                             # units of every shape there is, up to the largest
    assert [int(((lo < sizes) & (sizes <= hi)).sum()) >= 3 for lo, hi in ((0, 4096), (4096, 8192), (8192, 16384))] == [True] * 3
    assert 4096 in sizes and 8192 in sizes and sizes.max() <= 16384
