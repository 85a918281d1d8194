"""Enough tasks of the largest one-workgroup shape that the first workgroups start spread: against the CPU oracle, and what the
spread costs where it gains nothing (short tasks of the shape, many kernels)."""
import statistics
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding, traces
from parity_util import DEV, assert_profile_equal
from timing_util import below

pytestmark = pytest.mark.gpu


def tasks_of(rng, launches, ids):
    rec = np.zeros(sum(launches), dtype=traces.LAUNCH_DTYPE)
    n = rec.size
    rec["name_id"], rec["grid"], rec["block"] = rng.integers(0, ids, n) * 7919, 1, 64
    ex, gap = np.rint(rng.lognormal(9, 1, n)).astype(np.int64) + 1, np.rint(rng.lognormal(9, 1, n)).astype(np.int64)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    return rec, np.concatenate([[0], np.cumsum(launches)]).astype(np.uint64)


def repeated(rec, off, times):
    """The tasks `times` times over, on the GPU."""
    d_rec = binding.to_device_records(rec, DEV).repeat(times, 1)
    first = np.arange(times, dtype=np.uint64)[:, None] * off[-1]
    return d_rec, np.concatenate([(first + off[:-1]).ravel(), [off[-1] * times]]).astype(np.uint64)


@pytest.mark.parametrize("launches,times", [((8193, 8200, 9001, 16384), 256), ((8193, 8200, 9001, 16384), 255), ((12288, 700, 3, 16383, 5000), 1030)])
@pytest.mark.parametrize("ids", [20, 300])
def test_profiles_of_spread_tasks(launches, times, ids):
    rec, off = tasks_of(np.random.default_rng(ids), launches, ids)
    o_ids, o_rows, o_tro = oracle.profile(rec, off)
    d_rec, all_off = repeated(rec, off, times)
    rows = np.tile(o_rows, times)
    rows["task"] += np.repeat(np.arange(times, dtype=np.uint32) * len(launches), o_rows.size)
    tro = (np.arange(times, dtype=np.uint64)[:, None] * o_tro[-1] + o_tro[:-1]).ravel()
    prof = binding.fikit_profile(d_rec, binding.to_device_u64(all_off, DEV))
    assert_profile_equal(prof, np.tile(o_ids, times), rows, np.append(tro, o_tro[-1] * np.uint64(times)))


def test_spread_costs_nothing_where_it_gains_nothing():
    rec, off = tasks_of(np.random.default_rng(1), (8200,), 300)
    calls = {}
    for tasks in (1023, 1024):             # below the line, and on it
        d_rec, all_off = repeated(rec, off, tasks)
        d_off, n = binding.to_device_u64(all_off, DEV), int(all_off[-1])
        ids, row_off = (torch.empty(k, dtype=torch.int64, device=DEV) for k in (n, tasks + 1))
        rows = torch.empty((tasks * 300, 128), dtype=torch.uint8, device=DEV)
        ws = binding.workspace(binding.fikit_profile_workspace_bytes(n, tasks), DEV)
        calls[tasks] = lambda a=d_rec, b=d_off, c=ids, d=rows, e=row_off, f=ws: binding.fikit_profile(
            a, b, ids_out=c, rows_out=d, task_row_offsets_out=e, workspace_buf=f)

    def compare():
        took = {tasks: [] for tasks in calls}
        for _ in range(40):
            for tasks, call in calls.items():
                torch.cuda.synchronize()
                t = time.perf_counter()
                call()
                took[tasks].append((time.perf_counter() - t) / tasks)
        under, on = (statistics.median(took[tasks]) for tasks in calls)
        return on, 1.045 * under

    assert below(compare)                  # 1.01 with the spread by what the tasks are, 1.07 to 1.09 with one of the same length for all
