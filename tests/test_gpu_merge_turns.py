"""Merges whose tasks take the larger tables: more of them than there are workgroups, all or by list, checked against the CPU oracle;
and long tasks at the pace of fixed turns."""
import statistics
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding
from parity_util import DEV
from test_gpu_merge import check_merge
from timing_util import below

pytestmark = pytest.mark.gpu


def table(rng, sizes, step):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    n = int(off[-1])
    task = np.repeat(np.arange(len(sizes)), sizes)
    at = np.arange(n) - off[:-1].astype(np.int64)[task]
    rows = np.zeros(n, dtype=oracle.ROW_DTYPE)
    rows["kernel_id"], rows["task"] = at * 4 + step * (at % 3 == 0), task
    for blk in ("exec", "gap"):
        rows[blk]["count"] = rng.integers(1, 9, n)
        rows[blk]["sum"] = rng.integers(0, 2**62, n)
        for f in ("min", "max", "p50", "p95"):
            rows[blk][f] = rng.integers(0, 10**6, n)
    return rows, off


@pytest.mark.parametrize("large,small,rows", [(767, 0, 1040), (768, 0, 1040), (769, 0, 1040), (1600, 0, 1030), (800, 400, 1025), (1537, 900, 1030), (770, 300, 1)])
def test_more_tasks_than_workgroups(large, small, rows):
    rng = np.random.default_rng(large)
    sizes = rng.permutation(np.concatenate([np.full(large, rows), np.full(small, 2)]))
    a, b = table(rng, sizes, 0), table(rng, rng.permutation(np.where(sizes < 10, sizes, sizes % 7)), 1)
    check_merge(*a, *b)


def test_two_lengths_in_turn_cost_what_both_cost_apart():
    short, long, n = 100, 1800, 4000
    calls = {}
    for name, sizes in (("in turn", np.tile([short, long], n)), ("short", np.full(n, short)), ("long", np.full(n, long))):
        sides = []
        for step in (0, 1):
            off = np.concatenate([[0], np.cumsum(sizes)])
            task = torch.repeat_interleave(torch.arange(sizes.size, device=DEV), torch.from_numpy(sizes).to(DEV), output_size=int(off[-1]))
            d_off = torch.from_numpy(off).to(DEV)
            at = torch.arange(int(off[-1]), device=DEV) - d_off[task]
            rows = torch.ones((int(off[-1]), 16), dtype=torch.int64, device=DEV)
            rows[:, 0], rows[:, 1] = at * 4 + step * (at % 3 == 0), task
            sides += [rows.view(torch.uint8), d_off]
        out = torch.empty((2 * sides[0].shape[0], 128), dtype=torch.uint8, device=DEV)
        row_off = torch.empty(sizes.size + 1, dtype=torch.int64, device=DEV)
        ws = binding.workspace(binding.fikit_profile_merge_workspace_bytes(sizes.size), DEV)
        calls[name] = lambda s=sides, o=out, r=row_off, w=ws: binding.fikit_profile_merge(*s, rows_out=o, task_row_offsets_out=r, workspace_buf=w)

    def compare():
        took = {name: [] for name in calls}
        for _ in range(15):
            for name, call in calls.items():
                torch.cuda.synchronize()
                t = time.perf_counter()
                call()
                took[name].append(time.perf_counter() - t)
        us = {name: statistics.median(t) * 1e6 for name, t in took.items()}
        return us["in turn"], 1.2 * (us["short"] + us["long"])

    assert below(compare)                  # 0.92; 1.3 in fixed turns
