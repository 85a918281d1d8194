"""Per-launch measurements where a wave's lanes take each other's values: tasks, runs and the input's end at and around the wave's
last lane, overlapping launches, records that lie on 8 bytes only; against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding, traces
from parity_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1], [63], [64], [65], [62, 1, 1, 1], [64, 64], [0, 127, 0, 1, 0], [255, 257, 1], [300, 63, 65, 0]])
@pytest.mark.parametrize("run_of", [1000, 64, 63, 1])
@pytest.mark.parametrize("shift", [0, 8])
def test_measure_at_the_edges_of_waves(lens, run_of, shift):
    rng = np.random.default_rng(sum(lens) + run_of)
    n = sum(lens)
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = rng.integers(0, 9, n), 1, 64
    rec["start_ns"] = np.cumsum(rng.integers(0, 1 << 40, n))
    rec["end_ns"] = rec["start_ns"] + rng.integers(0, 1 << 41, n)      # some overlap the next launch
    rec["run"] = np.arange(n) // run_of
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    buf = torch.empty(64 * n + 16, dtype=torch.uint8, device=DEV)
    d_rec = buf[shift:shift + 64 * n].view(n, 64)
    d_rec.copy_(binding.to_device_records(rec, DEV).view(n, 64))
    assert d_rec.data_ptr() % 16 == shift
    ex, gap = binding.fikit_measure(d_rec, binding.to_device_u64(off, DEV))
    want = oracle.measure(rec, off)
    assert np.array_equal(ex.cpu().numpy(), want[0]) and np.array_equal(gap.cpu().numpy(), want[1])
