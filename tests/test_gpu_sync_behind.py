"""A device synchronisation behind a call finds the runtime done with the call: it takes about what it takes on an idle device."""
import statistics
import time

import pytest
import torch

from paper_2311_10359_amd import binding, traces
from timing_util import below

DEV = "cuda:0"

pytestmark = pytest.mark.gpu


def synchronisation_us():
    t = time.perf_counter()
    torch.cuda.synchronize()
    return (time.perf_counter() - t) * 1e6


@pytest.mark.parametrize("tasks,launches", [(2, 1000), (32, 30000)])
def test_nothing_is_left_behind_a_call(tasks, launches):
    cfg = traces.config(4, n_tasks=tasks, hp_launches=launches, lp_launches=launches)
    rec, off = traces.build(cfg, threads=4)
    hp, lp = traces.scenarios(cfg)
    d_rec, d_off = binding.to_device_records(rec, DEV), binding.to_device_u64(off, DEV)
    d_hp, d_lp, d_gaps = binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV), binding.to_device_u64(traces.gap_offsets(off, hp), DEV)

    def compare():
        idle, behind = [], []
        for _ in range(100):
            binding.fikit_profile_gapfill(d_rec, d_off, d_hp, d_lp, d_gaps, margin_ns=cfg.margin_ns, min_gap_ns=cfg.min_gap_ns)
            behind.append(synchronisation_us())
            idle.append(synchronisation_us())
        return statistics.median(behind), 2 * statistics.median(idle) + 2

    # 2.9 us on an idle device; 3.5 to 4.2 where the runtime was told or asked of the call's end, 12 to 32 where it was not
    assert below(compare)
