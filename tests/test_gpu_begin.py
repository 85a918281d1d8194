"""What precedes and follows the launches' own kernels: on both sides of the sizes from which on one workgroup no longer does it,
with rows that must not be written, and from several threads at once (needs an MI355X)."""
import threading

import numpy as np
import pytest
import torch

from paper_2311_10359_amd import binding, traces
from parity_util import DEV, check_gapfill, check_profile
from test_gpu_parity import ragged_trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tasks", [1, 1023, 1024, 2047, 2048, 2049, 8190, 8191, 8192, 20000])
@pytest.mark.parametrize("long_tasks", [0, 2])
def test_numbers_of_tasks_and_scenarios(n_tasks, long_tasks):
    rng = np.random.default_rng(n_tasks)
    lens = rng.integers(0, 9, n_tasks)
    lens[:min(3, n_tasks)] = [5000, 9000, 16384][:min(3, n_tasks)] if long_tasks else 700
    lens[n_tasks - min(long_tasks, n_tasks):] = 17001
    rec, off = ragged_trace(n_tasks, lens.tolist(), 7)
    print(f"{n_tasks} tasks, {rec.shape[0]} launches", flush=True)
    prof, d_off, o_prof = check_profile(rec, off)
    for n_scen in (1, 2048, 2049):
        hp, lp = (rng.integers(0, n_tasks, n_scen).astype(np.uint32) for _ in range(2))
        check_gapfill(prof, d_off, off, o_prof, hp, lp, 100, 0)


@pytest.mark.parametrize("n_tasks", [40, 2500])
def test_rows_of_a_refused_call_are_not_written(n_tasks):
    lens = np.full(n_tasks, 11)
    lens[3] = 20000
    rec, off = ragged_trace(5, lens.tolist(), 6)
    d_off = binding.to_device_u64(off, DEV)
    want = binding.fikit_profile(binding.to_device_records(rec, DEV), d_off)
    rows = torch.full((want.n_rows - 1, 128), 0x5a, dtype=torch.uint8, device=DEV)
    bad_rec = rec.copy()
    bad_rec["end_ns"][100] = bad_rec["start_ns"][100] - 1
    bad_off = off.copy()
    bad_off[7] = off[9] + 1
    for r, o, cap, status in ((rec, off, want.n_rows - 1, binding.FIKIT_ROW_CAPACITY), (bad_rec, off, want.n_rows - 1, binding.FIKIT_BAD_RECORD),
                              (rec, bad_off, want.n_rows - 1, binding.FIKIT_INVALID_ARG)):
        with pytest.raises(binding.FikitError) as e:
            binding.fikit_profile(binding.to_device_records(r, DEV), binding.to_device_u64(o, DEV), rows_out=rows, row_capacity=cap)
        assert e.value.status == status
        assert e.value.n_rows == (want.n_rows if status == binding.FIKIT_ROW_CAPACITY else 0)
        assert bool((rows == 0x5a).all())
    # the merge: too many rows, and offsets that rise past the rows there are before they fall back
    tro = want.task_row_offsets
    past = tro.clone()
    past[5] = want.n_rows + 3
    out = torch.full((want.n_rows - 1, 128), 0x5a, dtype=torch.uint8, device=DEV)
    for b_off, status in ((tro, binding.FIKIT_ROW_CAPACITY), (past, binding.FIKIT_INVALID_ARG)):
        with pytest.raises(binding.FikitError) as e:
            binding.fikit_profile_merge(want.rows, tro, want.rows, b_off, rows_out=out)
        assert e.value.status == status and bool((out == 0x5a).all())


def test_an_id_of_all_ones_without_a_row_is_unknown():
    """2^64 - 1 marks a free slot of the look-up tables: as a launch's ID it must not be found there."""
    rec, off = ragged_trace(3, [40, 50, 60], 5)
    prof, d_off, _ = check_profile(rec, off)
    hp, lp = np.array([0, 2], dtype=np.uint32), np.array([1, 1], dtype=np.uint32)
    d_hp, d_lp, d_go = binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV), binding.to_device_u64(traces.gap_offsets(off, hp), DEV)
    _, d_gap = binding.fikit_measure(binding.to_device_records(rec, DEV), d_off)
    lists = [binding.to_device_u64(np.array([0, 1, 2], dtype=np.uint64), DEV), d_lp, binding.to_device_u32(np.array([1, 2], dtype=np.uint32), DEV)]
    wide_lists = [binding.to_device_u64(np.array([0, 1, 71], dtype=np.uint64), DEV), binding.to_device_u32(np.full(71, 1, dtype=np.uint32), DEV),
                  binding.to_device_u32(np.full(71, 3, dtype=np.uint32), DEV)]
    for at in (3, 45):                                  # in a trace, in the queue
        ids = prof.ids.clone()
        ids[at] = -1
        args = (ids, d_off, prof.rows, prof.task_row_offsets)
        for call in (lambda: binding.fikit_gapfill(*args, d_hp, d_lp, d_go, margin_ns=0, min_gap_ns=0),
                     lambda: binding.fikit_gapfill_replay(*args, d_gap, d_hp, d_lp, d_go, margin_ns=0, min_gap_ns=0, feedback=True),
                     lambda: binding.fikit_prio_fill(*args, d_hp, *lists, d_go, margin_ns=0, min_gap_ns=0),
                     lambda: binding.fikit_prio_fill(*args, d_hp, *wide_lists, d_go, margin_ns=0, min_gap_ns=0)):
            with pytest.raises(binding.FikitError) as e:
                call()
            assert e.value.status == binding.FIKIT_UNKNOWN_ID


def test_calls_of_several_threads():
    rec, off = ragged_trace(9, [300, 20000, 5000, 1, 40], 12)
    want = binding.fikit_profile(binding.to_device_records(rec, DEV), binding.to_device_u64(off, DEV))
    wrong = []

    def work(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for cut in range(6):                       # every call has its own number of rows
                r, o = rec[: int(off[5 - (k + cut) % 5])], off[: 6 - (k + cut) % 5]
                d_rec, d_off = binding.to_device_records(r, DEV), binding.to_device_u64(o, DEV)
                got = binding.fikit_profile(d_rec, d_off)
                n = int(want.task_row_offsets[o.size - 1])
                if got.n_rows != n or not torch.equal(got.rows, want.rows[:n]):
                    wrong.append((k, cut, got.n_rows, n))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
