"""What a call returns is final when it returns: outputs can be read on any stream without a further wait, whether the host's own
look at the report sees the end of the call or the runtime's wait has to (a stream that is busy for several milliseconds first)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding, traces

DEV = "cuda:0"

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("busy_cycles", [0, 50_000, 20_000_000])
@pytest.mark.parametrize("own_stream", [False, True])
def test_results_are_final_on_return(busy_cycles, own_stream):
    cfg = traces.config(4, n_tasks=6, hp_launches=700, lp_launches=1100)
    rec, off = traces.build(cfg)
    rec["name_id"] += busy_cycles % 9973 + own_stream       # (no two cases have the same results)
    o_ids, o_rows, o_tro = oracle.profile(rec, off)
    hp, lp = traces.scenarios(cfg)
    gaps = traces.gap_offsets(off, hp)
    want = oracle.gapfill(o_ids, off, o_rows, o_tro, hp, lp, cfg.margin_ns, cfg.min_gap_ns, gaps)
    d_rec, d_off = binding.to_device_records(rec, DEV), binding.to_device_u64(off, DEV)
    d_hp, d_lp, d_gaps = binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV), binding.to_device_u64(gaps, DEV)
    kept = dict(rows_out=torch.empty((o_rows.size, 128), dtype=torch.uint8, device=DEV), ids_out=torch.empty(rec.size, dtype=torch.int64, device=DEV),
                task_row_offsets_out=torch.empty(off.size, dtype=torch.int64, device=DEV),
                out=binding.GapFill(torch.empty(int(gaps[-1]), dtype=torch.int32, device=DEV),
                                    *(torch.empty(k, dtype=torch.int64, device=DEV) for k in (int(gaps[-1]), hp.size, hp.size))))
    reader = torch.cuda.Stream()
    stream = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    torch.cuda.synchronize()
    for _ in range(3):
        # the outputs hold something else before the call
        for t in (kept["rows_out"], kept["ids_out"], kept["task_row_offsets_out"], *kept["out"]):
            t.fill_(0x5b)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            if busy_cycles:
                torch.cuda._sleep(busy_cycles)
            prof, out = binding.fikit_profile_gapfill(d_rec, d_off, d_hp, d_lp, d_gaps, margin_ns=cfg.margin_ns,
                                                      min_gap_ns=cfg.min_gap_ns)
        with torch.cuda.stream(reader):
            rows = prof.rows.to("cpu", non_blocking=True)
            filled, count = out.filled_ns.to("cpu", non_blocking=True), out.fill_count.to("cpu", non_blocking=True)
            done, placed = out.lp_completion_ns.to("cpu", non_blocking=True), out.lp_placed.to("cpu", non_blocking=True)
            reader.synchronize()
        assert rows.numpy().reshape(-1).tobytes()[:o_rows.nbytes] == o_rows.tobytes()
        assert prof.n_rows == o_rows.size
        assert np.array_equal(filled.numpy(), want[1]) and np.array_equal(count.numpy().view(np.uint32), want[0])
        assert np.array_equal(done.numpy(), want[2]) and np.array_equal(placed.numpy().view(np.uint64), want[3])
        torch.cuda.synchronize()
