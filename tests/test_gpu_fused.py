"""fikit_profile_gapfill (the two calls of the hot path as one) against the oracle: every output of the profile and of
the gap fill, bit for bit, where the profile's own kernels write the predictions (tasks that one workgroup holds) and where
they do not (long tasks, tasks left to the sort, predictions beyond 32 bits)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_10359_amd import binding, traces
from parity_util import DEV, LANES_MIN_SCENARIOS, assert_profile_equal, kernels_of
from test_gpu_parity import RAGGED_LENS, all_pairs, mixed_trace, ragged_trace

pytestmark = pytest.mark.gpu


def check_fused(rec, off, hp, lp, margin, min_gap, predictor=0, o_prof=None):
    o_ids, o_rows, o_tro = o_prof if o_prof is not None else oracle.profile(rec, off)
    go = traces.gap_offsets(off, hp)
    exp = oracle.gapfill(o_ids, off, o_rows, o_tro, hp, lp, margin, min_gap, go, predictor=predictor)
    prof, got = binding.fikit_profile_gapfill(binding.to_device_records(rec, DEV), binding.to_device_u64(off, DEV),
                                              binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV),
                                              binding.to_device_u64(go, DEV), margin_ns=margin, min_gap_ns=min_gap,
                                              predictor=predictor)
    torch.cuda.synchronize()
    assert_profile_equal(prof, o_ids, o_rows, o_tro)
    fc = binding.u32_to_numpy(got.fill_count)
    bad = np.nonzero(fc != exp[0])[0]
    assert bad.size == 0, f"fill_count differs at {bad[:5]}: {fc[bad[:5]]} vs {exp[0][bad[:5]]}"
    assert np.array_equal(got.filled_ns.cpu().numpy(), exp[1]), "filled_ns differs"
    assert np.array_equal(got.lp_completion_ns.cpu().numpy(), exp[2]), "lp_completion_ns differs"
    assert np.array_equal(binding.u64_to_numpy(got.lp_placed), exp[3]), "lp_placed differs"
    return (o_ids, o_rows, o_tro)


def test_batched_workload_shape():
    """The benchmark's shape at a reduced size: a high-priority trace and a low-priority queue per scenario (so few that a wave
    takes each); launches beyond 4096 and 8192 so that all three shapes of the task kernel write predictions."""
    for hp_l, lp_l in ((300, 1200), (4100, 8300)):
        cfg = traces.config(4, n_tasks=8400 if hp_l == 300 else 8200, hp_launches=hp_l, lp_launches=lp_l)
        rec, off = traces.build(cfg, threads=4)
        hp, lp = traces.scenarios(cfg)
        o = check_fused(rec, off, hp, lp, cfg.margin_ns, cfg.min_gap_ns)
        check_fused(rec, off, hp, lp, 0, 100000, predictor=binding.FIKIT_PREDICT_MEAN, o_prof=o)


def test_shared_tasks_in_both_roles():
    """Every ordered pair of 182 tasks (a task against itself included), which the lane walk takes: tasks are trace and queue at
    once."""
    cfg = traces.config(4, n_tasks=182, hp_launches=201, lp_launches=803)
    rec, off = traces.build(cfg, threads=4)
    hp, lp = all_pairs(range(cfg.n_tasks))
    assert hp.size >= LANES_MIN_SCENARIOS
    with kernels_of() as names:
        o = check_fused(rec, off, hp, lp, cfg.margin_ns, cfg.min_gap_ns)
    assert "k_gf_walk_lanes" in names and "k_gf_walk_wave" not in names
    check_fused(rec, off, hp, lp, 40000, 0, predictor=binding.FIKIT_PREDICT_MEAN, o_prof=o)


def test_mixed_task_shapes():
    """Every size class side by side, tasks with too many IDs for a workgroup, heavy ties: some tasks' predictions
    come from the profile's kernels, the others' from the gap fill's."""
    rec, off, lens = mixed_trace(21, 64, max_len=20000, wide=False)
    hp, lp = all_pairs(range(len(lens)))
    o = check_fused(rec, off, hp, lp, 100, 0)
    check_fused(rec, off, hp, lp, 0, 2000, predictor=binding.FIKIT_PREDICT_MEAN, o_prof=o)


def test_ragged_and_empty_tasks():
    lens = RAGGED_LENS
    rec, off = ragged_trace(4242, lens, 9)
    hp, lp = all_pairs(range(len(lens)))
    check_fused(rec, off, hp, lp, 300, 0)


def test_few_scenarios_and_none():
    """A few scenarios; no scenario: the profile."""
    cfg = traces.config(1, n_tasks=8, launches=3000)
    rec, off = traces.build(cfg, threads=4)
    hp, lp = traces.scenarios(cfg)
    check_fused(rec, off, hp, lp, cfg.margin_ns, cfg.min_gap_ns)
    none = np.zeros(0, dtype=np.uint32)
    check_fused(rec, off, none, none, 0, 0)


def test_predictions_beyond_32_bits():
    lens = [40 + k for k in range(64)]
    rec, off = ragged_trace(99, lens, 4)
    ex = (rec["end_ns"] - rec["start_ns"]).astype(np.int64)
    ex[rec["name_id"] == 1] += 5_000_000_000
    gp = np.full(rec.shape[0], 1000, dtype=np.int64)
    gp[rec["name_id"] == 2] = 6_000_000_000
    start = np.cumsum(ex + gp) - (ex + gp)
    rec["start_ns"] = start
    rec["end_ns"] = start + ex
    hp, lp = all_pairs(range(len(lens)))
    check_fused(rec, off, hp, lp, 300, 0)


def test_runs_and_errors():
    """A trace with run numbers (no idle time across runs) through the fused call; a bad record is reported."""
    cfg = traces.config(4, n_tasks=8400, hp_launches=64, lp_launches=96, runs=3)
    rec, off = traces.build(cfg, threads=4)
    hp, lp = traces.scenarios(cfg)
    check_fused(rec, off, hp, lp, cfg.margin_ns, cfg.min_gap_ns)
    bad = rec.copy()
    bad["end_ns"][5] = bad["start_ns"][5] - 1
    go = traces.gap_offsets(off, hp)
    with pytest.raises(binding.FikitError) as e:
        binding.fikit_profile_gapfill(binding.to_device_records(bad, DEV), binding.to_device_u64(off, DEV),
                                      binding.to_device_u32(hp, DEV), binding.to_device_u32(lp, DEV),
                                      binding.to_device_u64(go, DEV), margin_ns=0, min_gap_ns=0)
    assert e.value.status == -4


@pytest.mark.parametrize("n_tasks", [3, 1025, 2049])
@pytest.mark.parametrize("long_task", [False, True])
def test_the_fill_runs_ahead_of_the_host_only_behind_a_finished_profile(n_tasks, long_task):
    """The fill is enqueued before the host knows how the profile ended: it must leave its outputs alone where the rows do not fit
    or a record is bad, and be done again where a task was left to the sort."""
    rng = np.random.default_rng(n_tasks)
    lens = rng.integers(1, 40, n_tasks)
    lens[0], lens[1] = 3000, 17000 if long_task else 900
    rec, off = ragged_trace(11, lens.tolist(), 9)
    hp, lp = rng.integers(0, n_tasks, 50).astype(np.uint32), rng.integers(0, n_tasks, 50).astype(np.uint32)
    hp[0], lp[0], hp[1], lp[1] = 0, 1, 1, 0
    o = check_fused(rec, off, hp, lp, 100, 0)
    many = rec.copy()
    many["name_id"][:3000] = np.arange(3000)      # more IDs than a workgroup holds
    check_fused(many, off, hp, lp, 100, 0)
    go = traces.gap_offsets(off, hp)
    bad = rec.copy()
    bad["end_ns"][700] = bad["start_ns"][700] - 1
    for r, capacity, status in ((rec, len(o[1]) - 1, binding.FIKIT_ROW_CAPACITY), (bad, len(o[1]) + 8, binding.FIKIT_BAD_RECORD)):
        out = binding.GapFill(*(torch.full((k,), 77, dtype=d, device=DEV)
                                for k, d in ((int(go[-1]), torch.int32), (int(go[-1]), torch.int64), (50, torch.int64), (50, torch.int64))))
        with pytest.raises(binding.FikitError) as e:
            binding.fikit_profile_gapfill(binding.to_device_records(r, DEV), binding.to_device_u64(off, DEV), binding.to_device_u32(hp, DEV),
                                          binding.to_device_u32(lp, DEV), binding.to_device_u64(go, DEV), margin_ns=100, min_gap_ns=0,
                                          rows_out=torch.empty((capacity, 128), dtype=torch.uint8, device=DEV), out=out)
        assert e.value.status == status
        assert all(bool((x == 77).all()) for x in out)


@pytest.mark.parametrize("longest,launched", [(16384, False), (16385, True)])
def test_trace_names_the_look_ups_only_where_they_run(longest, launched):
    """The profile's kernels write the predictions of tasks that a workgroup holds; the look-ups run for longer ones."""
    rec, off = ragged_trace(2, [longest, 300, 160], 9)
    with kernels_of() as names:
        check_fused(rec, off, np.array([0, 1], dtype=np.uint32), np.array([1, 2], dtype=np.uint32), 100, 0)
    assert ("k_gf_predict32" in names) == launched
