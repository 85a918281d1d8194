"""The look-ups of predictions at the ends of what a workgroup and a lane read: tasks that start at odd and even places, IDs that lie
on 8 bytes only, with and without actual idle times; gap fill and replays against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2311_10359_amd import binding, traces
from parity_util import DEV, check_gapfill, check_profile
from test_gpu_replay import check_replay

pytestmark = pytest.mark.gpu


def trace(rng, lens, ids):
    n = sum(lens)
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = rng.integers(0, ids, n) * 7919, 1, 64
    ex, gap = rng.integers(1, 9000, n), rng.integers(0, 40000, n)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    return rec, np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)


@pytest.mark.parametrize("lens", [[1, 2, 3, 1], [511, 512, 513, 510], [1023, 1024, 1025, 1026, 1027, 1], [2047, 1, 2049, 3073, 4097, 2], [1, 9999, 8193, 16385]])
@pytest.mark.parametrize("shift", [0, 8])
@pytest.mark.parametrize("ids", [9, 600])        # (more kernels than the table in LDS holds: rows are searched in memory)
def test_lookups_at_the_ends_of_what_is_read(lens, shift, ids):
    rng = np.random.default_rng(sum(lens) + ids)
    rec, off = trace(rng, lens, ids)
    prof, d_off, o_prof = check_profile(rec, off)
    buf = torch.zeros(prof.ids.numel() * 8 + 16, dtype=torch.uint8, device=DEV)
    moved = buf[shift:shift + prof.ids.numel() * 8].view(torch.int64)
    moved.copy_(prof.ids)
    assert moved.data_ptr() % 16 == shift
    prof = prof._replace(ids=moved)
    tasks = len(lens)
    hp, lp = (a.ravel().astype(np.uint32) for a in np.meshgrid(np.arange(tasks), np.arange(tasks)))
    check_gapfill(prof, d_off, off, o_prof, hp, lp, 100, 0)
    d_gap = binding.fikit_measure(binding.to_device_records(rec, DEV), d_off)[1]
    check_replay(prof, d_off, off, o_prof, d_gap, d_gap.cpu().numpy(), hp, lp, 100, 0)
