"""fikit_gapfill_static with predictions beyond 32 bits, which it finds out on the device: scenarios that share tasks, a task that is
trace and queue at once, up to as many scenarios as take one launch and more, tasks of one launch; against the CPU oracle and fikit_gapfill."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding, traces
from parity_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tasks,n_scen,ids", [(2, 1, 5), (3, 9, 40), (12, 144, 30), (16, 256, 30), (17, 257, 8), (70, 4900, 8), (5, 25, 700)])
def test_static_with_long_predictions(n_tasks, n_scen, ids):
    rng = np.random.default_rng(n_tasks)
    lens = rng.integers(1, 3000 if ids > 100 else 600, n_tasks)
    lens[0] = 1
    n = int(lens.sum())
    rec = np.zeros(n, dtype=traces.LAUNCH_DTYPE)
    rec["name_id"], rec["grid"], rec["block"] = rng.integers(0, ids, n) * 7919, 1, 64
    ex, gap = rng.integers(1, 9000, n), rng.integers(0, 40000, n)
    rec["start_ns"] = np.cumsum(ex + gap) - (ex + gap)
    rec["end_ns"] = rec["start_ns"] + ex
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    o_ids, rows, tro = oracle.profile(rec, off)
    rows = rows.copy()
    for blk in ("exec", "gap"):
        rows[blk]["p50"] *= 1_000_003
    hp, lp = (a.ravel()[:n_scen].astype(np.uint32) for a in np.meshgrid(np.arange(n_tasks), np.arange(n_tasks)))
    gaps = traces.gap_offsets(off, hp)
    want = oracle.gapfill(o_ids, off, rows, tro, hp, lp, 500, 0, gaps)
    d_rows = torch.from_numpy(rows.view(np.uint8).reshape(-1, 128).copy()).to(DEV)
    args = (binding.to_device_u64(o_ids, DEV), binding.to_device_u64(off, DEV), d_rows, binding.to_device_u64(tro, DEV),
            binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV), binding.to_device_u64(gaps, DEV))
    n_gaps = int(gaps[-1])
    out = binding.GapFill(torch.full((n_gaps,), -7, dtype=torch.int32, device=DEV), *(torch.full((k,), -7, dtype=torch.int64, device=DEV)
                                                                                     for k in (n_gaps, n_scen, n_scen)))
    status = torch.full((1,), -99, dtype=torch.int32, device=DEV)
    for _ in range(2):
        binding.fikit_gapfill_static(*args, n_ids=n, n_gaps=n_gaps, margin_ns=500, min_gap_ns=0, out=out, status_out=status)
    torch.cuda.synchronize()
    assert int(status[0]) == binding.FIKIT_OK
    other = binding.fikit_gapfill(*args, margin_ns=500, min_gap_ns=0)
    for name, a, b, w in zip(out._fields, out, other, want):
        assert torch.equal(a, b), name
        assert np.array_equal(a.cpu().numpy().astype(np.int64), np.asarray(w).astype(np.int64)), name
