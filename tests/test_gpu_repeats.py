"""The walk where inputs repeat and results are copied: periods around the sizes of a block, a round and the shortest period that is
noted, traces and queues that stop repeating somewhere, a first pass unlike the others, queues that end inside a copied unit or never
move, by a workgroup per scenario and by a wave, against the CPU oracle.  Which ways through the search and the copy these inputs take
is checked in test_repeat_model.py."""
import numpy as np
import pytest

import oracle
from paper_2311_10359_amd import binding, traces
from parity_util import check_gapfill, check_profile, kernels_of
from repeat_model import LIMITS, follow
from test_gpu_replay import check_measure, check_replay

pytestmark = pytest.mark.gpu

# Up to so many scenarios, if their traces have so many launches on average, a workgroup takes each, otherwise a wave.  Repeats are looked
# for in traces of REPEAT_GAPS gaps and more.
TEAM_SCENARIOS, TEAM_LAUNCHES, REPEAT_GAPS = LIMITS["GF_TEAM_SCENARIOS"], LIMITS["GF_TEAM_LAUNCHES"], LIMITS["REPEAT_GAPS"]

WALKS, REPLAYS = {"k_gf_walk_wave", "k_gf_walk_team", "k_gf_walk_lanes"}, {"k_gf_replay_wave", "k_gf_replay_team", "k_gf_replay_lanes"}


def passes(rng, period, launches, ids, odd_at=(), first=0):
    """Kernel numbers of a task: `first` launches of their own, then passes of `period` launches; other kernels at the places odd_at."""
    order = rng.integers(0, ids, period)
    kid = np.concatenate([rng.integers(0, ids, first), np.resize(order, launches - first)]) if launches > first else rng.integers(0, ids, launches)
    for at in odd_at:
        if at < launches:
            kid[at] = ids + at % 3
    return kid


def tasks_of(rng, kids, exec_of, gap_of):
    """Records in which a kernel number has one duration and one idle time (the predictions are these values)."""
    kid = np.concatenate(kids)
    rec = np.zeros(kid.size, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"] = kid
    rec["grid"], rec["block"] = 1, 64
    e, g = exec_of[kid], gap_of[kid]
    rec["start_ns"] = np.cumsum(e + g) - (e + g)
    rec["end_ns"] = rec["start_ns"] + e
    return rec, np.concatenate([[0], np.cumsum([k.size for k in kids])]).astype(np.uint64)


def grid(times, team):
    """Traces and queues in all pairs: kernel numbers of the tasks, durations and idle times, high- and low-priority tasks."""
    rng = np.random.default_rng(sum(map(ord, times)))
    ids = 23
    exec_of, gap_of = rng.integers(100, 4000, ids + 3), rng.integers(0, 3000, ids + 3)
    if times == "many":
        exec_of = rng.integers(10, 300, ids + 3)
    elif times == "stuck":
        exec_of[::4] = 1 << 20
    elif times == "zeros":
        exec_of[::2], gap_of[::3] = 0, 0
        gap_of *= 2
    elif times == "wide_sums":
        exec_of, gap_of = exec_of << 19, np.minimum(4 * gap_of, 8191) << 19
    hp = [passes(rng, p, n, ids, odd, first) for p, n, odd, first in (
        (1, 2500, (), 0), (2, 2900, (600,), 0), (7, 4097, (), 0), (63, REPEAT_GAPS, (), 0), (64, REPEAT_GAPS + 1, (), 0),
        (65, REPEAT_GAPS + 2, (1300, 1301), 0), (127, 3000, (), 0), (128, 3000, (2999,), 0), (129, 3000, (2998,), 0), (200, 5000, (), 0), (200, 5000, (900, 2100, 3300, 4400), 0),
        (255, 2500, (), 0), (256, 2561, (1280,), 0), (257, 2571, (), 0), (600, 6000, (), 300), (200, 8000, (5000,), 2300), (3000, 5900, (), 0), (7, 0, (), 0), (7, 1, (), 0))]
    lp = [passes(rng, p, n, ids, odd, 0) for p, n, odd in (
        (1, 5000, ()), (13, 3000, ()), (63, 6000, ()), (160, 9000, ()), (160, 9000, (700, 3000)), (160, 400, ()), (161, 1000, (999,)), (64, 64, ()),
        (600, 9000, ()), (4000, 4000, ()), (1, 1, ()), (1, 0, ()))]
    if team:   # (a trace that alone brings the average there)
        hp.append(passes(rng, 50, TEAM_LAUNCHES * (len(hp) + 1), ids))
    h, l = (a.ravel().astype(np.uint32) for a in np.meshgrid(range(len(hp)), range(len(hp), len(hp) + len(lp)), indexing="ij"))
    return hp + lp, exec_of, gap_of, h, l


def stops(team):
    """One trace of kernels that are all different, long enough for many repeats, and queues of which one entry differs: inside the fourth
    unit that is compared, its last one, the one behind it; passes so long that places repeat only after the period has been doubled; one
    that never repeats.  The same with a trace that stops repeating soon, and with one that goes on repeating behind a launch.  As grid()."""
    rng, ids, n = np.random.default_rng(3), 200, 30000
    exec_of, gap_of = rng.integers(1000, 12000, ids + 3), rng.integers(0, 30000, ids + 3)
    whole, queue = np.resize(rng.permutation(ids), n), passes(rng, 160, 3 * n, ids)
    rec, off = tasks_of(rng, [whole, queue], exec_of, gap_of)
    o_ids, o_rows, o_tro = oracle.profile(rec, off)
    pair = np.array([0], np.uint32), np.array([1], np.uint32)
    counts = oracle.gapfill(o_ids, off, o_rows, o_tro, *pair, 0, 0, traces.gap_offsets(off, pair[0]))[0]
    a, ja, D, dq = follow(gap_of[whole], exec_of[queue], counts, team)[1]

    def but_for(kid, at):
        kid = kid.copy()
        kid[at] = ids
        return kid

    odd, late = but_for(whole, a + 5 * D + 3), but_for(whole, n // 2)
    queues = [queue] + [but_for(queue, ja + at) for at in (3 * dq + dq // 2, 4 * dq - 1, 4 * dq)]
    queues += [passes(rng, 6007, 3 * n, ids), passes(rng, 7001, 3 * n, ids), rng.integers(0, ids, 3 * n)]
    kids = [whole, odd, late] + queues
    h, l = np.repeat([0, 1, 2], len(queues)), np.tile(3 + np.arange(len(queues)), 3)
    if not team:   # (short scenarios, which bring the average down to the walk by wave)
        kids.append(np.resize(whole, 100))
        h, l = (np.concatenate([x, np.full(3 * x.size, len(kids) - 1)]) for x in (h, l))
    return kids, exec_of, gap_of, h.astype(np.uint32), l.astype(np.uint32)


@pytest.mark.parametrize("times", ["few", "many", "stuck", "zeros", "wide_sums", "stops"])
@pytest.mark.parametrize("team", [True, False])
def test_what_repeats_is_copied(times, team):
    kids, exec_of, gap_of, h, l = stops(team) if times == "stops" else grid(times, team)
    rec, off = tasks_of(np.random.default_rng(1), kids, exec_of, gap_of)
    prof, d_off, o_prof = check_profile(rec, off)
    assert h.size <= TEAM_SCENARIOS
    d_gap, gap = check_measure(rec, off)
    for copies, margin, min_gap in ((1, 0, 0), (1, 50, 500)) + ((-(-(TEAM_SCENARIOS + 1) // h.size), 20, 0),) * (not team):
        hs, ls = np.tile(h, copies), np.tile(l, copies)
        print(f"{hs.size} scenarios, {times}, margin {margin}", flush=True)
        with kernels_of() as names:
            check_gapfill(prof, d_off, off, o_prof, hs, ls, margin, min_gap)
        assert names & WALKS == {"k_gf_walk_team" if team else "k_gf_walk_wave"}
        with kernels_of() as names:
            check_replay(prof, d_off, off, o_prof, d_gap, gap, hs, ls, margin, min_gap)
        assert names & REPLAYS == {"k_gf_replay_team" if team else "k_gf_replay_wave"}


# Tasks that no scenario uses do not count: neither a long one beside short scenarios nor short ones beside long scenarios.
@pytest.mark.parametrize("n_scen,launches,unused,team", [
    (TEAM_SCENARIOS, TEAM_LAUNCHES, [], True), (TEAM_SCENARIOS + 1, TEAM_LAUNCHES, [], False),
    (3, TEAM_LAUNCHES, [], True), (3, TEAM_LAUNCHES - 1, [], False),
    (3, 100, [3 * TEAM_LAUNCHES], False), (3, TEAM_LAUNCHES, [100] * 40, True)])
def test_a_workgroup_takes_a_scenario_while_all_fit(n_scen, launches, unused, team):
    rng = np.random.default_rng(launches)
    rec, off = tasks_of(rng, [passes(rng, 200, launches, 20), passes(rng, 160, launches, 20)] + [passes(rng, 50, n, 20) for n in unused],
                        rng.integers(100, 4000, 23), rng.integers(0, 3000, 23))
    prof, d_off, o_prof = check_profile(rec, off)
    d_gap, gap = check_measure(rec, off)
    hs, ls = np.zeros(n_scen, np.uint32), np.ones(n_scen, np.uint32)
    with kernels_of() as names:
        check_gapfill(prof, d_off, off, o_prof, hs, ls, 0, 0)
        check_replay(prof, d_off, off, o_prof, d_gap, gap, hs, ls, 0, 0)
    assert names & (WALKS | REPLAYS) == ({"k_gf_walk_team", "k_gf_replay_team"} if team else {"k_gf_walk_wave", "k_gf_replay_wave"})


def walk_ms(prof, d_off, off, o_prof, hs, ls):
    """Least time of the walk of a gap fill in four calls, whose results are checked."""
    ms = []
    for _ in range(4):
        binding.fikit_trace_enable(True)
        try:
            check_gapfill(prof, d_off, off, o_prof, hs, ls, 0, 0)
            times = binding.fikit_trace_read()
        finally:
            binding.fikit_trace_enable(False)
        ms += [t for name, (t, _) in times.items() if name in WALKS]
    assert len(ms) == 4
    return min(ms)


@pytest.mark.parametrize("team", [True, False])
def test_what_repeats_is_not_walked(team):
    """A trace that repeats, one that does but for a launch in every 15,000, and one that does not: copying shows in the time (measured:
    0.29, 3.5 and 7.9 ms by a workgroup, 0.88, 3.6 and 7.6 by a wave; 0.98 and 0.63 of the first two are copied).  Short scenarios beside
    them bring the average down to the walk by wave."""
    rng, n, ids = np.random.default_rng(11), 120000, 200
    e, g = rng.integers(1000, 12000, ids + 3), rng.integers(0, 30000, ids + 3)
    order = rng.permutation(ids)
    whole = np.resize(order, n)
    odd = whole.copy()
    odd[15000::15000] = ids + np.arange(odd[15000::15000].size) % 3
    short = np.resize(order, 100)
    kids = [whole, odd, rng.permutation(whole), passes(rng, 160, 3 * n, ids), short]
    rec, off = tasks_of(rng, kids, e, g)
    prof, d_off, o_prof = check_profile(rec, off)
    few = 0 if team else 40
    ms = []
    for trace in (0, 1, 2):
        hs, ls = np.array([trace] * 4 + [4] * few, np.uint32), np.array([3] * 4 + [4] * few, np.uint32)
        ms.append(walk_ms(prof, d_off, off, o_prof, hs, ls))
    print(f"walk in ms: {ms}", flush=True)
    assert ms[0] < 0.4 * ms[2] and ms[1] < 0.6 * ms[2], ms
