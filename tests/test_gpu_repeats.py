"""The walk where inputs repeat and results are copied: periods around the sizes of a block, a round and the shortest period that is
noted, traces and queues that stop repeating somewhere, a first pass unlike the others, queues that end inside a copied unit or never
move, by a workgroup per scenario and by a wave, against the CPU oracle."""
import numpy as np
import pytest

from paper_2311_10359_amd import binding, traces
from parity_util import check_gapfill, check_profile, kernels_of
from repeat_model import follow
from test_gpu_replay import check_measure, check_replay

pytestmark = pytest.mark.gpu

# Up to so many scenarios, if they have so many gaps on average, a workgroup takes each, otherwise a wave.  Repeats are looked
# for in traces of REPEAT_GAPS gaps and more.
TEAM_SCENARIOS, TEAM_GAPS, REPEAT_GAPS = 768, 16384, 2048

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


@pytest.mark.parametrize("times", ["few", "many", "stuck", "zeros", "wide_sums"])
@pytest.mark.parametrize("team", [True, False])
def test_what_repeats_is_copied(times, team):
    rng = np.random.default_rng(sum(map(ord, times)))
    ids = 23
    exec_of, gap_of = rng.integers(100, 4000, ids + 3), rng.integers(0, 3000, ids + 3)
    if times == "many":
        exec_of = rng.integers(10, 300, ids + 3)
    elif times == "stuck":
        exec_of[::4] = 1 << 20
    elif times == "zeros":
        exec_of[::2], gap_of[::3] = 0, 0
    elif times == "wide_sums":
        exec_of, gap_of = exec_of << 19, gap_of << 19
    hp = [passes(rng, p, n, ids, odd, first) for p, n, odd, first in (
        (1, 2500, (), 0), (2, 2900, (600,), 0), (7, 4097, (), 0), (63, REPEAT_GAPS, (), 0), (64, REPEAT_GAPS + 1, (), 0),
        (65, REPEAT_GAPS + 2, (1300, 1301), 0), (127, 3000, (), 0), (128, 3000, (2999,), 0), (129, 3000, (2998,), 0), (200, 5000, (), 0), (200, 5000, (900, 2100, 3300, 4400), 0),
        (255, 2500, (), 0), (256, 2561, (1280,), 0), (257, 2571, (), 0), (600, 6000, (), 300), (200, 8000, (5000,), 2300), (3000, 5900, (), 0))]
    lp = [passes(rng, p, n, ids, odd, 0) for p, n, odd in (
        (1, 5000, ()), (13, 3000, ()), (63, 6000, ()), (160, 9000, ()), (160, 9000, (700, 3000)), (160, 400, ()), (161, 1000, (999,)), (64, 64, ()),
        (600, 9000, ()), (4000, 4000, ()), (1, 1, ()))]
    if team:   # (a trace that alone brings the average there)
        hp.append(passes(rng, 50, TEAM_GAPS * (len(hp) + 1) + 1, ids))
    rec, off = tasks_of(rng, hp + lp, exec_of, gap_of)
    prof, d_off, o_prof = check_profile(rec, off)
    h, l = (a.ravel().astype(np.uint32) for a in np.meshgrid(range(len(hp)), range(len(hp), len(hp) + len(lp)), indexing="ij"))
    assert h.size <= TEAM_SCENARIOS < 6 * h.size
    d_gap, gap = check_measure(rec, off)
    for copies, margin, min_gap in ((1, 0, 0), (1, 50, 500)) + ((6, 20, 0),) * (not team):
        hs, ls = np.tile(h, copies), np.tile(l, copies)
        print(f"{hs.size} scenarios, {times}, margin {margin}", flush=True)
        with kernels_of() as names:
            check_gapfill(prof, d_off, off, o_prof, hs, ls, margin, min_gap)
        assert names & WALKS == {"k_gf_walk_team" if team else "k_gf_walk_wave"}
        with kernels_of() as names:
            check_replay(prof, d_off, off, o_prof, d_gap, gap, hs, ls, margin, min_gap)
        assert names & REPLAYS == {"k_gf_replay_team" if team else "k_gf_replay_wave"}


# Tasks that no scenario uses do not count: neither a long one beside short scenarios nor short ones beside long scenarios.
@pytest.mark.parametrize("n_scen,gaps,unused,team", [
    (TEAM_SCENARIOS, TEAM_GAPS, [], True), (TEAM_SCENARIOS + 1, TEAM_GAPS, [], False),
    (3, TEAM_GAPS, [], True), (3, TEAM_GAPS - 1, [], False),
    (3, 100, [3 * TEAM_GAPS], False), (3, TEAM_GAPS, [100] * 40, True)])
def test_a_workgroup_takes_a_scenario_while_all_fit(n_scen, gaps, unused, team):
    rng = np.random.default_rng(gaps)
    rec, off = tasks_of(rng, [passes(rng, 200, gaps + 1, 20), passes(rng, 160, gaps + 1, 20)] + [passes(rng, 50, n, 20) for n in unused],
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
