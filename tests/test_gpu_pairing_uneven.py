"""Pairing searches in which scenarios differ a lot in their gaps, or all of a task's tie: against the CPU oracle, and what they take
beside even ones."""
import statistics
import time

import numpy as np
import pytest
import torch

from paper_2311_10359_amd import binding
from parity_util import DEV
from test_gpu_pairing import check_pairing
from timing_util import below

pytestmark = pytest.mark.gpu
WAVES = 8192                  # from this many scenarios on a wave takes one, in rounds of as many


def with_gaps(rng, gaps, n_tasks):
    n = gaps.size
    off = np.concatenate([[0], np.cumsum(gaps)]).astype(np.uint64)
    return (rng.integers(0, n_tasks, n).astype(np.uint32), rng.integers(0, n_tasks, n).astype(np.uint32), n_tasks, off,
            rng.integers(-2**40, 2**40, int(off[-1])), rng.integers(0, 2**40, n))


@pytest.mark.parametrize("n_scen,base,longs,length", [
    (WAVES, 3, [0], 8192), (WAVES, 3, [0], 8193), (WAVES, 1500, [1, 2, 3, 8191], 12001), (WAVES, 1500, [1, 2, 3, 8191], 20001),
    (WAVES + 5, 0, [4, 5, 8192, 8196], 50000), (2 * WAVES, 10, list(range(0, 2 * WAVES, 40)), 9000),
    (65 * WAVES + 3, 0, [r * WAVES + w for r in range(66) for w in (0, 1, 2)] + [r * WAVES + 3 for r in range(65)], 8193),   # more than a workgroup lists
])
def test_few_scenarios_of_many_gaps(n_scen, base, longs, length):
    rng = np.random.default_rng(length)
    gaps = rng.integers(0, 2 * base + 1, n_scen)
    gaps[longs] = length
    check_pairing(*with_gaps(rng, gaps, 300))


@pytest.mark.parametrize("n_scen", [9, 255, 257, 5000, 8192, 30000])
@pytest.mark.parametrize("tasks", [[0], list(range(64)), [511], list(range(600)), [5 + 512 * k for k in range(12)]])   # (the last: one place in a table for all)
@pytest.mark.parametrize("order", ["falling", "rising", "mixed", "equal", "extreme"])
def test_scenarios_that_tie(n_scen, tasks, order):
    rng = np.random.default_rng(n_scen)
    comp = {"falling": np.arange(n_scen)[::-1], "rising": np.arange(n_scen), "mixed": rng.permutation(n_scen), "equal": np.zeros(n_scen),
            "extreme": np.where(np.arange(n_scen) < n_scen - 2, 2**63 - 1, -2**63)}[order].astype(np.int64)
    gaps = rng.integers(0, 3, n_scen)
    off = np.concatenate([[0], np.cumsum(gaps)]).astype(np.uint64)
    filled = np.zeros(int(off[-1]), dtype=np.int64)
    hp = np.asarray(tasks, dtype=np.uint32)[np.arange(n_scen) % len(tasks) if order == "mixed" else rng.integers(0, len(tasks), n_scen)]
    check_pairing(hp, rng.integers(0, 600, n_scen).astype(np.uint32), max(600, max(tasks) + 1), off, filled, comp)


def took_us(calls):
    took = [[] for _ in calls]
    for _ in range(25):
        for call, us in zip(calls, took):
            torch.cuda.synchronize()
            t = time.perf_counter()
            call()
            us.append((time.perf_counter() - t) * 1e6)
    return [statistics.median(us) for us in took]


def call_of(gaps, comp, filled_up_to):
    n = gaps.size
    off = np.concatenate([[0], np.cumsum(gaps)]).astype(np.uint64)
    d_off, d_task = binding.to_device_u64(off, DEV), torch.zeros(n, dtype=torch.int32, device=DEV)
    filled = torch.randint(0, filled_up_to, (int(off[-1]),), device=DEV)
    d_comp = torch.from_numpy(np.ascontiguousarray(comp, dtype=np.int64)).to(DEV)
    ws = binding.workspace(binding.fikit_pairing_workspace_bytes(1), DEV)
    return lambda: binding.fikit_pairing_best(d_task, d_task, 1, d_off, filled, d_comp, workspace_buf=ws)


def test_one_long_scenario_costs_the_same_among_more_others():
    gaps = np.full(WAVES, 1000)
    gaps[7] = 1_000_000
    calls = [call_of(gaps, np.arange(WAVES), 1000), call_of(gaps[:-1], np.arange(WAVES - 1), 1000)]     # by waves, by workgroups

    def compare():
        waves, workgroups = took_us(calls)
        return waves, 1.3 * workgroups

    assert below(compare)                  # 1.02; 2.2 by waves alone


def test_order_of_tied_scenarios_does_not_matter():
    gaps = np.full(2 * WAVES, 3)
    calls = [call_of(gaps, np.arange(gaps.size)[::-1], 1), call_of(gaps, np.zeros(gaps.size), 1)]       # falling completions, equal ones

    def compare():
        falling, equal = took_us(calls)
        return falling, 1.4 * equal

    assert below(compare)                  # 1.0; 1.65 to 2.2 if all of them try
