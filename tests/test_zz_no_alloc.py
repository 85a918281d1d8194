"""fikit_gapfill_static (the gap fill on the library's built-in scratch buffer, for callers that cannot allocate)
against fikit_gapfill, bit for bit, through the C ABI: two calls in a row, the second on a smaller input, so that
what the first call left in the shared scratch buffer must not show in the second."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2311_10359_amd import binding, traces
from test_gpu_parity import all_pairs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_both(cfg, margin, min_gap, predictor=binding.FIKIT_PREDICT_P50, pairs=traces.scenarios):
    rec, off = traces.build(cfg, threads=4)
    d_off = binding.to_device_u64(off, DEV)
    prof = binding.fikit_profile(binding.to_device_records(rec, DEV), d_off)
    hp, lp = pairs(cfg)
    go = traces.gap_offsets(off, hp)
    d_hp, d_lp, d_go = binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV), binding.to_device_u64(go, DEV)
    want = binding.fikit_gapfill(prof.ids, d_off, prof.rows, prof.task_row_offsets, d_hp, d_lp, d_go, margin_ns=margin,
                                 min_gap_ns=min_gap, predictor=predictor)
    n_gaps, s = int(go[-1]), hp.size
    # outputs pre-filled with a pattern: every element must be overwritten
    got = binding.GapFill(torch.full((n_gaps,), -7, dtype=torch.int32, device=DEV),
                          torch.full((n_gaps,), -7, dtype=torch.int64, device=DEV),
                          torch.full((s,), -7, dtype=torch.int64, device=DEV),
                          torch.full((s,), -7, dtype=torch.int64, device=DEV))
    status = torch.full((1,), -99, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    binding.fikit_gapfill_static(prof.ids, d_off, prof.rows, prof.task_row_offsets, d_hp, d_lp, d_go, n_ids=int(off[-1]),
                                 n_gaps=n_gaps, margin_ns=margin, min_gap_ns=min_gap, predictor=predictor, out=got,
                                 status_out=status)
    assert torch.cuda.memory_allocated() == before          # (torch's allocator was not asked for anything)
    torch.cuda.synchronize()
    assert int(status[0]) == binding.FIKIT_OK
    for a, b, name in zip(got, want, binding.GapFill._fields):
        assert torch.equal(a, b), f"{name} differs from fikit_gapfill"
    return int(want.lp_placed.sum())


def test_two_calls_in_a_row_the_second_smaller():
    # 4096 scenarios of 64 + 190 launches = 1,040,384 launches
    big = traces.config(4, n_tasks=8192, hp_launches=64, lp_launches=190)
    small = traces.config(4, n_tasks=40, hp_launches=500, lp_launches=1500)
    assert run_both(big, 500, 0) > 0
    assert run_both(small, 500, 0) > 0
    # so many scenarios that a lane takes each
    all_of = traces.config(4, n_tasks=182, hp_launches=101, lp_launches=403)
    assert run_both(all_of, 500, 0, pairs=lambda cfg: all_pairs(range(cfg.n_tasks))) > 0
    assert run_both(small, 500, 0) > 0
    # few scenarios sharing traces (one wave per scenario), the paper's 0.1 ms threshold, the mean predictor
    grid = traces.config(1, n_tasks=8, launches=20000)
    run_both(grid, 500, 100000)
    run_both(small, 0, 0, predictor=binding.FIKIT_PREDICT_MEAN)


def test_limits_and_device_side_status():
    lib = binding.load()
    p = binding._GapfillParams(500, 0, 0, 0)
    fake, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(None)

    def call(n_ids, n_tasks):
        return lib.fikit_gapfill_static(fake, n_ids, fake, n_tasks, fake, fake, fake, fake, 1, ctypes.byref(p), fake, 1, fake,
                                        fake, fake, fake, fake, null)
    assert call(binding.FIKIT_STATIC_MAX_IDS + 1, 2) == binding.FIKIT_TOO_LARGE
    assert call(1000, binding.FIKIT_STATIC_MAX_TASKS + 1) == binding.FIKIT_TOO_LARGE
    assert binding.status_string(binding.FIKIT_TOO_LARGE) not in ("ok", "unknown status")
    # a wrong n_gaps is found on the device and reported through the status word
    cfg = traces.config(4, n_tasks=8, hp_launches=100, lp_launches=300)
    rec, off = traces.build(cfg)
    d_off = binding.to_device_u64(off, DEV)
    prof = binding.fikit_profile(binding.to_device_records(rec, DEV), d_off)
    hp, lp = traces.scenarios(cfg)
    go = traces.gap_offsets(off, hp)
    n_gaps, s = int(go[-1]), hp.size
    out = binding.GapFill(torch.zeros(n_gaps + 8, dtype=torch.int32, device=DEV), torch.zeros(n_gaps + 8, dtype=torch.int64, device=DEV),
                          torch.zeros(s, dtype=torch.int64, device=DEV), torch.zeros(s, dtype=torch.int64, device=DEV))
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    binding.fikit_gapfill_static(prof.ids, d_off, prof.rows, prof.task_row_offsets, binding.to_device_u32(hp, DEV),
                                 binding.to_device_u32(lp, DEV), binding.to_device_u64(go, DEV), n_ids=int(off[-1]),
                                 n_gaps=n_gaps + 1, margin_ns=500, min_gap_ns=0, out=out, status_out=status)
    torch.cuda.synchronize()
    assert int(status[0]) == binding.FIKIT_INVALID_ARG
