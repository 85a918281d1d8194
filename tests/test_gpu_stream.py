"""Long tasks in which a few Kernel IDs are so frequent that no workgroup holds all their launches: every output of the
profile against the CPU oracle, and whether the sort was needed."""
import numpy as np
import pytest

import oracle
from paper_2311_10359_amd import traces
from parity_util import check_profile, kernels_of

pytestmark = pytest.mark.gpu
LONG = 1 << 18      # tasks from this length on are not sorted for a frequent ID


def skewed(seed, lens, n_ids, heavy, times):
    """Tasks of the given lengths; a launch is kernel 0 with probability `heavy`, else one of n_ids."""
    rng = np.random.default_rng(seed)
    n = sum(lens)
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    kid = np.where(rng.random(n) < heavy, 0, rng.integers(0, n_ids, n)).astype(np.uint32)
    rec["name_id"], rec["grid"], rec["block"] = kid * 7919, 1, 64
    if times == "lognormal":
        ex = np.maximum(1, np.rint(rng.lognormal(8.5 + (kid % 5), 1.5, n))).astype(np.int64)
        gp = np.where(rng.random(n) < 0.3, 0, np.rint(rng.lognormal(9.6, 1.2, n))).astype(np.int64)
    elif times == "ties":
        ex, gp = np.full(n, 12345, np.int64), (kid % 3).astype(np.int64)
    elif times == "wide":           # the whole range of 32 bits, clustered at both ends
        ex = np.where(rng.random(n) < 0.5, rng.integers(0, 9, n), (1 << 32) - 2 - rng.integers(0, 9, n)).astype(np.int64)
        gp = (np.int64(1) << rng.integers(0, 32, n)) - rng.integers(0, 2, n)
    else:                           # one value in a thousand beyond 32 bits
        ex = rng.integers(1, 100000, n) + np.where(rng.random(n) < 0.001, 1 << 33, 0)
        gp = rng.integers(0, 1000, n)
    start = np.cumsum(ex + gp) - (ex + gp)
    rec["start_ns"], rec["end_ns"] = start, start + ex
    rec["run"] = np.arange(n) // 100003
    off = np.zeros(len(lens) + 1, dtype=np.uint64)
    np.cumsum(lens, out=off[1:])
    return rec, off


@pytest.mark.parametrize("lens,n_ids,heavy,times,sorts", [
    ([LONG], 1, 1.0, "lognormal", False),                        # one ID, the shortest such task
    ([LONG + 1, 17, LONG + 4095], 3, 0.9, "ties", False),
    ([LONG - 1], 40, 0.5, "lognormal", True),                    # one launch shorter: sorted
    ([16385, 5000, LONG + 777, 300], 90, 0.3, "wide", False),    # beside tasks of every other shape
    ([500000, 600, 300001], 4096, 0.2, "lognormal", False),
    ([700001], 60000, 0.4, "lognormal", True),                   # more IDs in a bucket than its table holds
    ([300000, 900, 290000], 30000, 0.4, "lognormal", True),      # ... in the buckets beside it only
    ([4100000], 100000, 0.1, "ties", True),                      # ... in it, not in the ones beside it
    ([LONG, LONG], 50, 0.5, "beyond", True),
])
def test_frequent_ids(lens, n_ids, heavy, times, sorts):
    print(f"lengths {lens}, {n_ids} IDs, share of the first {heavy}, {times}", flush=True)
    rec, off = skewed(len(lens) + n_ids, lens, n_ids, heavy, times)
    with kernels_of() as names:
        check_profile(rec, off)
    assert ("k_onesweep_pass" in names) == sorts, sorted(names)


def with_rare(seed, tasks):
    """Tasks of (launches, frequent IDs, IDs launched once to `most` times): the frequent ones about equally often, the rare ones
    at random places and at the task's last launches."""
    rng = np.random.default_rng(seed)
    lens = [n for n, _, _, _ in tasks]
    kids = []
    for t, (n, frequent, rare, most) in enumerate(tasks):
        kid = rng.integers(0, frequent, n)
        times = rng.integers(1, most + 1, rare)
        at = rng.choice(n, int(times.sum()), replace=False)
        kid[at] = np.repeat(frequent + np.arange(rare), times)
        if rare:
            kid[-1] = frequent + rare - 1
        kids.append(kid + 100_000 * t)
    kid = np.concatenate(kids).astype(np.uint32)
    n = kid.size
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = kid * 7919, 1, 64
    ex = np.maximum(1, np.rint(rng.lognormal(8.5, 1.0, n))).astype(np.int64) + kid % 97
    gp = np.rint(rng.lognormal(9.0, 1.0, n)).astype(np.int64)
    rec["start_ns"] = np.cumsum(ex + gp) - (ex + gp)
    rec["end_ns"] = rec["start_ns"] + ex
    off = np.zeros(len(lens) + 1, dtype=np.uint64)
    np.cumsum(lens, out=off[1:])
    return rec, off


def sorted_with(rec, off):
    """Compares the profile with the oracle's; was a task sorted?"""
    with kernels_of() as names:
        check_profile(rec, off)
    return "k_onesweep_pass" in names


@pytest.mark.parametrize("tasks", [
    [(4_300_000, 30, 40, 1), (900, 100, 0, 1)],                       # more tiles than a unit can list: all buckets are streamed,
    [(900, 100, 0, 1), (4_300_000, 100, 300, 20)],                    # also those of a single launch (here behind a short task's)
    [(50_000, 10, 5, 1)],                                             # a bucket of one launch between two of which neither
    [(100_000, 20, 5, 1), (20_000, 40, 9, 2), (700, 30, 0, 1)],       # can take it in
    [(131_072, 30, 5, 1), (131_073, 30, 5, 1)],
    [(1_000_000, 20, 5, 1), (300_000, 3, 200, 15)],                   # ... beside streamed ones
])
def test_rare_ids_beside_frequent_ones(tasks):
    """Buckets with more rows than their launches would leave room for: the rows' room is the task's, nothing is sorted."""
    print(f"tasks {tasks}", flush=True)
    assert not sorted_with(*with_rare(len(tasks) + tasks[0][0], tasks))


def test_more_rows_than_the_task_has_room_for():
    """Nine units of 256 IDs each in 16,644 launches: 2304 rows, room for 2080.  The task is sorted."""
    names = np.arange(400_000, dtype=np.uint32)
    rec = np.zeros(names.size, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = names, 1, 64
    top = oracle.profile(rec, np.array([0, names.size], dtype=np.uint64))[0] >> np.uint64(56)
    kid = []
    for unit, launches in enumerate([256, 3841] * 4 + [256]):
        mine = names[top == 20 * unit + 3][:256]
        assert mine.size == 256
        kid.append(np.resize(mine, launches))
    kid = np.random.default_rng(3).permutation(np.concatenate(kid))
    rec = np.zeros(kid.size, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = kid, 1, 64
    rec["start_ns"] = np.arange(kid.size) * 1000
    rec["end_ns"] = rec["start_ns"] + 1 + kid % 997
    assert sorted_with(rec, np.array([0, kid.size], dtype=np.uint64))


def test_more_tiles_than_a_unit_can_list():
    """A task of more than 1024 tiles: all of its buckets are streamed, large and small."""
    rec, off = skewed(5, [4_200_000, 900], 300, 0.1, "lognormal")
    check_profile(rec, off)


def names_by_bucket(n=400_000):
    """Kernel names (their number) by the bucket that their IDs fall into."""
    names = np.arange(n, dtype=np.uint32)
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = names, 1, 64
    top = oracle.profile(rec, np.array([0, n], dtype=np.uint64))[0] >> np.uint64(56)
    return [names[top == b] for b in range(256)]


def trace_of(kids, ex, gap):
    """One task per array of kernel names."""
    kid = np.concatenate(kids)
    rec = np.zeros(kid.size, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = kid, 1, 64
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    return rec, np.concatenate([[0], np.cumsum([k.size for k in kids])]).astype(np.uint64)


@pytest.mark.parametrize("ids,sorts", [(512, False), (600, True)])
def test_task_that_a_large_unit_gives_up_while_it_is_streamed(ids, sorts):
    """A bucket of 12,000 launches holds as many IDs as its unit's table, or more; another bucket of the task is streamed beside it."""
    by, rng = names_by_bucket(), np.random.default_rng(ids)
    assert by[9].size >= ids
    others = np.concatenate([by[b][:1] for b in range(0, 256, 3) if b not in (6, 9)])
    kids = [rng.permutation(np.concatenate([np.full(230_000, by[6][0]), np.resize(by[9][:ids], 12_000), rng.choice(others, 58_000)]))
            for _ in range(3)]
    n = sum(k.size for k in kids)
    rec, off = trace_of(kids, np.maximum(1, np.rint(rng.lognormal(8.5, 1.5, n))).astype(np.int64), rng.integers(0, 30_000, n))
    assert sorted_with(rec, off) == sorts


def by_turn(kid):
    """How often each launch's kernel has been launched before it."""
    order = np.argsort(kid, kind="stable")
    first = np.r_[0, np.flatnonzero(np.diff(kid[order])) + 1]
    turn = np.empty(kid.size, dtype=np.int64)
    turn[order] = np.arange(kid.size) - np.repeat(first, np.diff(np.r_[first, kid.size]))
    return turn


def crowded(rng, launches, kind):
    """A task of LONG launches whose bucket 30 holds one ID per entry of `launches`; IDs of other buckets fill it up."""
    by = names_by_bucket()
    others = np.concatenate([by[b][:1] for b in range(0, 256, 2) if b != 30])
    rest = LONG + 5 - sum(launches)
    kid = rng.permutation(np.concatenate([np.repeat(by[30][:len(launches)], launches), rng.choice(others, rest - 1)]))
    kid = np.append(kid, others[:1])                         # (the task's last launch, which has no idle time)
    if kind == "lognormal":
        ex = np.maximum(1, np.rint(rng.lognormal(9 + kid % 5, 0.3 + 0.4 * (kid % 4)))).astype(np.int64)
        return trace_of([kid], ex, ex[::-1])
    # nearly all of an ID's values lie in one bin between its least and its largest
    turn = by_turn(kid)
    v = np.where(turn == 0, 10, np.where(turn == 1, 4_000_000_000, 1_000_000 + turn * 6151 % 200_000))
    return trace_of([kid], v, v)


@pytest.mark.parametrize("kind", ["lognormal", "clustered"])
@pytest.mark.parametrize("launches", [
    [40_000] + [2048, 2049, 3000, 4095, 4096, 4097, 2048, 5000, 33, 1],      # few IDs with as many bins as there can be
    [20_000] * 12,
    [30_000] + [33] * 255,                                                   # as many IDs as the table holds, with short lists ...
    [30_000] + [20 + i % 44 for i in range(255)],                            # ... and with some too long for one
    [17_000] + [300] * 255,
])
def test_streamed_bucket_wants_more_room_than_there_is(launches, kind):
    """The bins that a streamed bucket's IDs want do not fit their 24,576 words; clustered, the bins of the second round do not
    either, nor the lists of 31 samples each (255 IDs of 33 launches: 1020 lists of 32 words): the largest are cut to fit."""
    log2_above = lambda n: int(n - 1).bit_length()
    assert 2 * sum(1 << min(11, log2_above(n)) for n in launches) > 24576 and sum(launches) > 16384
    rec, off = crowded(np.random.default_rng(len(launches)), launches, kind)
    with kernels_of() as names:
        _, _, (ids, _, _) = check_profile(rec, off)
    assert "k_onesweep_pass" not in names, sorted(names)
    in_30 = ids[ids >> np.uint64(56) == 30]
    assert np.unique(in_30).size == len(launches) and in_30.size == sum(launches)
