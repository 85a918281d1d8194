"""The walks of the priority-queue fill where their windows begin and end and on both sides of the rule that picks one: queues
one launch shorter and longer than a window, many equal durations, levels shared and not, against the CPU oracle."""
import numpy as np
import pytest

from parity_util import check_profile
from test_gpu_prio import check_prio, prio_lists
from test_gpu_walk import trace_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_max", [1, 2, 3, 4, 7, 9, 16])
@pytest.mark.parametrize("n_scen", [333, 24600])
def test_prio_walk_edges(k_max, n_scen):
    lens = [0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 66]
    if n_scen < 1000:
        lens += [127, 128, 129, 130, 191, 192, 193, 400]
    for seed, (execs, gaps) in enumerate([([100, 250], [0, 90, 400, 900]), ([0, 1, 7, 7], [0, 3, 40]),
                                          ([1 << 31, (1 << 32) - 2, 5], [0, 9, 1 << 31, (1 << 32) - 2])]):
        rec, off = trace_of(10 * k_max + seed, lens, execs, gaps)
        prof, d_off, o_prof = check_profile(rec, off)
        for same_level in (0.1, 0.9):
            hp, lo, lt, lq = prio_lists(np.random.default_rng(seed), len(lens), n_scen, k_max, same_level)
            print(f"{n_scen} scenarios, up to {k_max} tasks, durations {execs}, same level {same_level}", flush=True)
            check_prio(prof, d_off, off, o_prof, hp, lo, lt, lq, 3, 5)
