"""The walks of the gap fill and of the replay where their windows begin and end: queues and traces one launch shorter and longer
than a window, gaps that take several windows, and running sums of the queue that pass 32 bits, against the CPU oracle."""
import numpy as np
import pytest

from paper_2311_10359_amd import traces
from parity_util import LANES_MIN_SCENARIOS, check_gapfill, check_profile, kernels_of
from test_gpu_parity import all_pairs
from test_gpu_prio import check_prio
from test_gpu_replay import check_measure, check_replay

pytestmark = pytest.mark.gpu


def trace_of(seed, lens, exec_choices, gap_choices):
    """Tasks whose Kernel IDs have one duration and one idle time each (so the predictions are these values)."""
    rng = np.random.default_rng(seed)
    total = int(sum(lens))
    rec = np.zeros(total, dtype=traces.LAUNCH_DTYPE)
    kid = rng.integers(0, 8, total)
    rec["name_id"] = kid
    rec["grid"], rec["block"] = 1, 64
    ex = np.asarray(rng.choice(exec_choices, 8), dtype=np.int64)[kid]
    gp = np.asarray(rng.choice(gap_choices, 8), dtype=np.int64)[kid]
    rec["start_ns"] = np.cumsum(ex + gp) - (ex + gp)
    rec["end_ns"] = rec["start_ns"] + ex
    off = np.zeros(len(lens) + 1, dtype=np.uint64)
    np.cumsum(lens, out=off[1:])
    return rec, off


@pytest.mark.parametrize("exec_choices,gap_choices", [
    ([100, 250], [0, 90, 400, 900]),                            # a few kernels per gap
    ([1], [0, 62, 63, 64, 200]),                                # whole windows per gap
    ([0, 1, 7], [0, 3, 40]),                                    # kernels without duration
    ([1 << 31, (1 << 32) - 2, 5], [0, 9, 1 << 31, (1 << 32) - 2]),   # running sums past 32 bits
    ([1 << 26, 3 << 25, 1], [1 << 27, 1 << 30, 2]),             # ... after many launches
])
@pytest.mark.parametrize("copies", [1, 3, 7])                   # 676 and 6084 scenarios: a wave each; 33,124: a lane each
def test_walk_edges(exec_choices, gap_choices, copies):
    lens = [1, 2, 3, 8, 15, 16, 17, 31, 32, 33, 61, 62, 63, 64, 65, 125, 126, 127, 128, 129, 189, 190, 255, 256, 257, 700] * copies
    rec, off = trace_of(copies + len(gap_choices), lens, exec_choices, gap_choices)
    prof, d_off, o_prof = check_profile(rec, off)
    hp, lp = all_pairs(range(len(lens)))
    with kernels_of() as names:
        for margin, min_gap in ((0, 0), (3, 50)):
            print(f"{hp.size} scenarios, durations {exec_choices}, margin {margin}", flush=True)
            check_gapfill(prof, d_off, off, o_prof, hp, lp, margin, min_gap)
    walks = names & {"k_gf_walk_lanes", "k_gf_walk_wave"}
    assert walks == {"k_gf_walk_lanes" if hp.size >= LANES_MIN_SCENARIOS else "k_gf_walk_wave"}
    d_gap, gap = check_measure(rec, off)
    check_replay(prof, d_off, off, o_prof, d_gap, gap, hp, lp, 3, 0)


@pytest.mark.parametrize("n_scen,launches", [(2048, 40000), (2049, 8 * 2049 - 1), (2049, 8 * 2049), (2049, 16 * 2049), (5000, 90000), (32767, 8 * 32767)])
def test_walk_order(n_scen, launches):
    """Waves take the scenarios by buckets of their traces' lengths: below and from the number of scenarios on from which they do, with
    lists that just fit and that do not, traces of no launch to a few thousand, and all of one bucket."""
    rng = np.random.default_rng(n_scen + launches)
    share = np.exp(rng.uniform(0, 6, 300))
    lens = (0.9 * launches * share / share.sum()).astype(np.int64)
    lens[:4] = 0, 1, 16, 17
    lens[-1] += launches - lens.sum()
    rec, off = trace_of(n_scen, list(lens), [100, 250], [0, 90, 400, 900])
    prof, d_off, o_prof = check_profile(rec, off)
    few = np.flatnonzero(lens < 3000)
    hp, lp = rng.choice(few, n_scen).astype(np.uint32), rng.choice(few, n_scen).astype(np.uint32)
    with kernels_of() as names:
        check_gapfill(prof, d_off, off, o_prof, hp, lp, 3, 0)
    assert "k_gf_walk_wave" in names
    d_gap, gap = check_measure(rec, off)
    check_replay(prof, d_off, off, o_prof, d_gap, gap, hp, lp, 3, 0)
    check_gapfill(prof, d_off, off, o_prof, np.full(n_scen, hp[0]), lp, 3, 0)
    if n_scen <= 12288:
        entries = np.arange(n_scen + 1, dtype=np.uint64) * 2
        both = np.stack([lp, rng.choice(few, n_scen).astype(np.uint32)], axis=1).ravel()
        check_prio(prof, d_off, off, o_prof, hp, entries, both, np.full(2 * n_scen, 3, dtype=np.uint32), 3, 0)
