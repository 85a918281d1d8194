"""The walks of the priority-queue fill where their windows begin and end and on both sides of the rule that picks one: queues
one launch shorter and longer than a window, many equal durations, levels shared and not, against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2311_10359_amd import binding, traces
from parity_util import DEV, check_profile, kernels_of
from test_gpu_prio import check_prio, prio_lists
from test_gpu_walk import trace_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_max", [1, 2, 3, 4, 7, 9, 16])
@pytest.mark.parametrize("n_scen", [333, 24600])
def test_prio_walk_edges(k_max, n_scen):
    lens = [0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 66]
    if n_scen < 1000:
        lens += [127, 128, 129, 130, 191, 192, 193, 400]
    for seed, (execs, gaps) in enumerate([([100, 250], [0, 90, 400, 900]), ([0, 1, 7, 7], [0, 3, 40]),
                                          ([1 << 31, (1 << 32) - 2, 5], [0, 9, 1 << 31, (1 << 32) - 2])]):
        rec, off = trace_of(10 * k_max + seed, lens, execs, gaps)
        prof, d_off, o_prof = check_profile(rec, off)
        for same_level in (0.1, 0.9):
            hp, lo, lt, lq = prio_lists(np.random.default_rng(seed), len(lens), n_scen, k_max, same_level)
            print(f"{n_scen} scenarios, up to {k_max} tasks, durations {execs}, same level {same_level}", flush=True)
            check_prio(prof, d_off, off, o_prof, hp, lo, lt, lq, 3, 5)


@pytest.mark.parametrize("k_max", [1, 2, 3, 7, 16])
def test_prio_groups_of_lanes_on_long_queues(k_max):
    """So many scenarios that a group of lanes takes each: queues that pass through the kernel's rings many times, traces whose
    results do too, result buffers off a 16-byte boundary."""
    lens = [0, 1, 17, 64, 95, 127, 128, 129, 191, 257, 311, 400, 513]
    rec, off = trace_of(k_max, lens, [100, 250, 40], [0, 90, 900, 4000])
    prof, d_off, o_prof = check_profile(rec, off)
    hp, lo, lt, lq = prio_lists(np.random.default_rng(k_max), len(lens), 24600, k_max, 0.5)
    n_gaps = int(traces.gap_offsets(off, hp)[-1])
    out = binding.PrioFill(torch.empty(n_gaps + 1, dtype=torch.int32, device=DEV)[1:],
                           torch.empty(n_gaps + 1, dtype=torch.int64, device=DEV)[1:],
                           torch.empty(lt.size, dtype=torch.int64, device=DEV), torch.empty(lt.size, dtype=torch.int64, device=DEV))
    with kernels_of() as names:
        for buffers in (None, out):
            print(f"{hp.size} scenarios of up to {k_max} tasks, {n_gaps} gaps", flush=True)
            check_prio(prof, d_off, off, o_prof, hp, lo, lt, lq, 3, 5, out=buffers)
    assert "k_pf_walk" in names and "k_pf_walk_wave" not in names


@pytest.mark.parametrize("n_scen", [1024, 1025])
@pytest.mark.parametrize("k", [2, 3, 5, 16])
def test_prio_levels_of_one_or_two_requests(n_scen, k):
    """Both sides of the number of scenarios up to which such levels are gone through in scalars."""
    lens = [0, 1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 200]
    rec, off = trace_of(k, lens, [100, 250, 250, 40], [0, 90, 400, 2000])
    prof, d_off, o_prof = check_profile(rec, off)
    rng = np.random.default_rng(k)
    hp = rng.integers(0, len(lens), n_scen).astype(np.uint32)
    lo = np.arange(n_scen + 1, dtype=np.uint64) * k
    lt = rng.integers(0, len(lens), n_scen * k).astype(np.uint32)
    lq = np.concatenate([1 + rng.permutation(k) // 2 for _ in range(n_scen)]).astype(np.uint32)
    check_prio(prof, d_off, off, o_prof, hp, lo, lt, lq, 3, 5)


@pytest.mark.parametrize("n_scen,lists,rare,walk,listed", [
    (2048, 1, 1, "wave", False), (2049, 1, 1, "wave", True),
    (24576, 1, 1, "wave", True), (24577, 1, 1, "lanes", False),
    (12288, 3, 3, "wave", True), (12289, 3, 3, "lanes", False), (12289, 9, 9, "wave", True),
    (12289, 1, 3, "lanes", True), (12289, 3, 9, "wave", False),      # the widest scenario is not like the others
])
def test_prio_order_is_made_where_waves_walk(n_scen, lists, rare, walk, listed):
    """Scenarios are listed by their traces' lengths for walks that read the lists, as far as the average scenario tells."""
    lens = [0, 1, 2, 16, 17, 24, 40] + [14_000] * 32               # (the long ones make room for the lists; nobody uses them)
    rec, off = trace_of(n_scen, lens, [100, 250, 40], [0, 90, 900])
    prof, d_off, o_prof = check_profile(rec, off)
    rng = np.random.default_rng(n_scen)
    k = np.full(n_scen, lists)
    k[5] = rare
    k[10:10 + rare - lists] -= 1                                    # (as many entries on average as the others have)
    lo = np.concatenate([[0], np.cumsum(k)]).astype(np.uint64)
    hp, lt = rng.integers(0, 7, n_scen).astype(np.uint32), rng.integers(0, 7, int(lo[-1])).astype(np.uint32)
    lq = rng.integers(1, 10, int(lo[-1])).astype(np.uint32)
    with kernels_of() as names:
        got, _ = check_prio(prof, d_off, off, o_prof, hp, lo, lt, lq, 3, 5)
    assert ("k_pf_walk_wave" in names) == (walk == "wave") and ("k_pf_walk" in names) == (walk == "lanes")
    ws = torch.zeros(binding.fikit_prio_fill_workspace_bytes(rec.size, len(lens), n_scen), dtype=torch.uint8, device=DEV)
    again = binding.fikit_prio_fill(prof.ids, d_off, prof.rows, prof.task_row_offsets, binding.to_device_u32(hp, DEV),
                                    binding.to_device_u64(lo, DEV), binding.to_device_u32(lt, DEV), binding.to_device_u32(lq, DEV),
                                    binding.to_device_u64(traces.gap_offsets(off, hp), DEV), margin_ns=3, min_gap_ns=5, workspace_buf=ws)
    assert all(torch.equal(a, b) for a, b in zip(again, got))
    counts = ws[:256].view(torch.int32)[20:52]                      # (behind the control block: scenarios on each list)
    assert int(counts.sum()) == (n_scen if listed else 0)
