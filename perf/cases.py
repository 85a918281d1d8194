"""Workloads of this library as a user's program runs them, for timing and comparing builds.

A case names an entry point of the binding (`path`) and the sizes of its inputs.  Inputs are drawn on the GPU with the
structure that `paper_2311_10359_amd/traces.py` draws on the host: a task repeats a pass over its kernels (`pass`), or
draws them uniformly or by Zipf's law; a kernel has a characteristic duration and idle time with lognormal scatter;
some idle times are long stalls, some are zero.  Tasks 0 .. hp_tasks-1 are traces of the high-priority service, the
lp_tasks behind them queues of the low-priority one; with `ragged` the lengths of a group's tasks are spread from 1 to
twice `*_launches` (odd numbers among them), otherwise all are `*_launches` long.

All outputs are whole numbers and have to be equal.
"""
import math

import numpy as np
import torch

from paper_2311_10359_amd import binding

DEV = "cuda:0"
LN = math.log
CHUNK = 1 << 23                       # launches drawn at a time
MOST_LAUNCHES = 1 << 27               # of a drawn case
GOLDEN = 0.6180339887498949


def _case(path, **sizes):
    """A case with every field: what is not named is the ordinary choice."""
    case = {
        "path": path,
        "hp_tasks": 1, "hp_launches": 4096, "hp_ids": 100,
        "lp_tasks": 0, "lp_launches": 16384, "lp_ids": 80,
        "ragged": False,
        "pattern": "pass",             # pass | uniform | zipf
        "hp_exec_ns": 20000.0, "hp_exec_sigma": 0.8, "hp_gap_ns": 30000.0, "hp_gap_sigma": 1.2,
        "lp_exec_ns": 6000.0, "lp_exec_sigma": 1.0, "lp_gap_ns": 8000.0, "lp_gap_sigma": 1.0,
        "stalls": 0.0,                 # share of idle times that are stalls of about 0.2 ms
        "zero_gaps": 0.0,              # share of launches that follow back to back
        "runs": 1,                     # measured runs a task's trace is made of
        "scenarios": 0,
        "lists": 1,                    # prio: low-priority tasks per scenario
        "mean": False,                 # predictor: mean instead of median
        "min_gap_ns": 0,
        "feedback": False,             # replay
        "want_ids": True,              # profile: the Kernel IDs are an output
    }
    assert set(sizes) <= set(case), sorted(set(sizes) - set(case))
    case.update(sizes)
    return case


def listed():
    small_pass = dict(hp_gap_ns=8000.0, hp_gap_sigma=1.0, lp_exec_ns=20000.0, lp_exec_sigma=0.8)
    return [
        # one service pair, one scenario: what an online scheduler asks for when a task has been measured; all latency
        dict(_case("step", hp_tasks=1, lp_tasks=1, hp_launches=1000, lp_launches=1000, hp_ids=20, lp_ids=15, scenarios=1,
                   **small_pass), name="tiny_step"),
        # the gap fill inside a serving loop: no allocation, no synchronisation, many calls in a row, odd lengths
        dict(_case("static", hp_tasks=8, lp_tasks=8, hp_launches=1501, lp_launches=3001, scenarios=64), name="static_serving"),
        # every pair of 16 + 16 long traces, a tenth of the idle times stalls: few scenarios of many gaps
        dict(_case("step", hp_tasks=16, lp_tasks=16, hp_launches=65536, lp_launches=65536, hp_ids=300, lp_ids=300,
                   scenarios=256, stalls=0.1, **small_pass), name="medium_step"),
        # the flagship workload (a quarter of it, so that several inputs fit the card): many independent scenarios
        dict(_case("step", hp_tasks=16384, lp_tasks=16384, scenarios=16384), name="batched_step"),
        # statistics only, few kernels carry most launches: long segments
        dict(_case("profile", hp_tasks=64, hp_launches=1 << 20, hp_ids=4096, pattern="zipf", zero_gaps=0.3, hp_exec_ns=5000.0,
                   hp_exec_sigma=1.5, hp_gap_ns=15000.0), name="skewed_profile"),
        # statistics only, the largest set of records
        dict(_case("profile", hp_tasks=256, hp_launches=1 << 20, hp_ids=1000, pattern="uniform", hp_gap_ns=8000.0,
                   hp_gap_sigma=1.0), name="large_profile"),
        # the gap fill on a profile at hand, predicted by means, tasks of all lengths from one launch on
        dict(_case("gapfill", hp_tasks=6000, lp_tasks=5000, hp_launches=1400, lp_launches=5200, scenarios=6000, ragged=True,
                   mean=True), name="ragged_gapfill"),
        # the per-launch measurements of traces of several runs
        dict(_case("measure", hp_tasks=6001, hp_launches=4000, ragged=True, runs=5), name="ragged_measure"),
        # the plan replayed against what happened, with feedback
        dict(_case("replay", hp_tasks=6000, lp_tasks=6000, hp_launches=2048, lp_launches=8192, scenarios=6000, feedback=True),
             name="replay_feedback"),
        # several low-priority services wait at different priorities
        dict(_case("prio", hp_tasks=4096, lp_tasks=4096, hp_launches=1024, lp_launches=2048, scenarios=4096, lists=3),
             name="prio_three"),
        # the best partner among all pairs of 128 + 128 services
        dict(_case("pairing", hp_tasks=128, lp_tasks=128, hp_launches=2048, lp_launches=4096, scenarios=16384), name="pairing_grid"),
        # a further run's profile merged into the profile so far
        dict(_case("merge", hp_tasks=20000, hp_launches=900, hp_ids=90), name="merge_runs"),
    ]


def _between(rng, lo, hi):
    """A whole number from lo to hi, even over its logarithm."""
    return int(round(math.exp(rng.uniform(LN(lo), LN(hi)))))


def draw(rng):
    path = rng.choice(("step", "step", "step", "profile", "profile", "gapfill", "static", "measure", "replay", "prio", "pairing",
                       "merge"))
    case = _case(path, ragged=rng.random() < 0.4, mean=rng.random() < 0.3, min_gap_ns=rng.choice((0, 0, 0, 5000)),
                 hp_gap_ns=rng.choice((8000.0, 15000.0, 30000.0)), hp_gap_sigma=rng.choice((1.0, 1.2)))
    if path in ("profile", "measure"):
        # a few long traces to many short ones
        case["hp_tasks"] = _between(rng, 1, 20000)
        case["hp_launches"] = _between(rng, 64, 1 << 20)
        case["runs"] = rng.choice((1, 1, 3))
        case["pattern"] = rng.choice(("pass", "uniform", "zipf"))
        case["hp_ids"] = _between(rng, 10, 4096 if case["pattern"] == "zipf" else 1000)
        case["zero_gaps"] = rng.choice((0.0, 0.3))
        case["hp_exec_sigma"] = rng.choice((0.8, 1.0, 1.5))
        case["want_ids"] = rng.random() < 0.8
        most = MOST_LAUNCHES
    elif path == "merge":
        case["hp_tasks"] = _between(rng, 16, 20000)
        case["hp_ids"] = _between(rng, 10, 2000)
        case["hp_launches"] = 10 * case["hp_ids"]
        most = MOST_LAUNCHES // 4
    elif path == "static":
        case["hp_tasks"], case["lp_tasks"] = _between(rng, 1, 64), _between(rng, 1, 64)
        case["hp_launches"], case["lp_launches"] = _between(rng, 64, 4096), _between(rng, 64, 4096)
        case["scenarios"] = max(case["hp_tasks"], min(case["hp_tasks"] * case["lp_tasks"], _between(rng, 1, 1024)))
        most = 1 << 19
    else:
        grid = rng.random() < 0.4      # every pair of a few services, or a queue for every trace
        case["hp_launches"], case["lp_launches"] = _between(rng, 100, 16384), _between(rng, 100, 16384)
        case["hp_ids"], case["lp_ids"] = _between(rng, 10, 300), _between(rng, 10, 300)
        case["stalls"] = rng.choice((0.0, 0.1))
        if grid:
            case["hp_tasks"], case["lp_tasks"] = _between(rng, 2, 96), _between(rng, 2, 96)
            case["scenarios"] = case["hp_tasks"] * case["lp_tasks"]
        else:
            case["hp_tasks"] = _between(rng, 1, 16384)
            case["lp_tasks"] = max(1, case["hp_tasks"] - rng.choice((0, case["hp_tasks"] // 3)))
            case["scenarios"] = case["hp_tasks"]
        case["feedback"] = path == "replay" and rng.random() < 0.6
        case["lists"] = rng.choice((2, 3, 4, 6, 9)) if path == "prio" else 1
        most = MOST_LAUNCHES // (16 if path == "prio" else 1)

    def size(c):
        return max(c["hp_tasks"] * c["hp_launches"] + c["lp_tasks"] * c["lp_launches"],
                   c["scenarios"] * (c["hp_launches"] + c["lists"] * c["lp_launches"] // 2 if c["lp_tasks"] else c["hp_launches"]))

    while size(case) > most:           # fewer tasks, then shorter ones
        if case["hp_tasks"] > 64:
            case["hp_tasks"] = case["hp_tasks"] * 2 // 3
            case["lp_tasks"] = case["lp_tasks"] * 2 // 3
        else:
            case["hp_launches"] = max(64, case["hp_launches"] * 2 // 3)
            case["lp_launches"] = max(64, case["lp_launches"] * 2 // 3)
        if case["scenarios"]:
            case["scenarios"] = max(case["hp_tasks"], min(case["scenarios"], case["hp_tasks"] * case["lp_tasks"]) * 2 // 3)
    if case["scenarios"] > case["hp_tasks"] * case["lp_tasks"]:
        case["scenarios"] = case["hp_tasks"] * case["lp_tasks"]
    return case


# ---- the shape of a case (no GPU needed) ----------------------------------------------------------------------------

def _lengths(tasks, launches, ragged):
    if not ragged:
        return np.full(tasks, launches, dtype=np.int64)
    return 1 + np.floor(2 * launches * np.modf((np.arange(tasks) + 1) * GOLDEN)[0]).astype(np.int64)


def _groups(case):
    hp = _lengths(case["hp_tasks"], case["hp_launches"], case["ragged"])
    lp = _lengths(case["lp_tasks"], case["lp_launches"], case["ragged"])
    return hp, lp


def _offsets(lengths):
    return np.concatenate([np.zeros(1, np.int64), np.cumsum(lengths)])


def _scenarios(case):
    """(hp_task, lp_task, gap_offsets) on the host: every pair of services, or the queues dealt to the traces in turn."""
    s = np.arange(case["scenarios"], dtype=np.int64)
    hp = s * case["hp_tasks"] // max(1, case["scenarios"])
    lp = case["hp_tasks"] + s % max(1, case["lp_tasks"])
    h = _groups(case)[0][hp]
    return hp, lp, _offsets(np.maximum(h - 1, 0))


def _row_bound(case):
    hp, lp = _groups(case)
    return int(np.minimum(hp, case["hp_ids"]).sum() + np.minimum(lp, case["lp_ids"]).sum())


def work(case):
    """Bytes that a pass cannot do without: every input read once, every output written once."""
    hp, lp = _groups(case)
    launches, tasks = int(hp.sum() + lp.sum()), hp.size + lp.size
    rows = 128 * _row_bound(case)
    _, _, gaps = _scenarios(case)
    fill = 12 * int(gaps[-1]) + 32 * case["scenarios"]
    path = case["path"]
    if path == "measure":
        total = (64 + 16) * launches + 8 * tasks
    elif path == "profile":
        total = (64 + 8 * case["want_ids"]) * launches + rows + 16 * tasks
    elif path == "step":
        total = 72 * launches + rows + 16 * tasks + fill
    elif path in ("gapfill", "static"):
        total = 8 * launches + rows + 16 * tasks + fill
    elif path == "replay":
        total = 8 * launches + 8 * int(hp.sum()) + rows + 16 * tasks + fill
    elif path == "prio":
        total = 8 * launches + rows + 16 * tasks + fill + 24 * case["scenarios"] * case["lists"]
    elif path == "pairing":
        total = 8 * int(gaps[-1]) + 32 * case["scenarios"] + 20 * tasks
    else:
        total = 3 * rows + 24 * tasks
    return {"bytes": int(total), "flops": 0}


def tolerance(case):
    return "exact"


# ---- inputs ------------------------------------------------------------------------------------------------------------

def _characters(gen, tasks, ids, exec_ns, exec_sigma, gap_ns, gap_sigma):
    """What a group of tasks keeps from run to run: per (task, ID) the launch tuple and the typical log times, per task the order
    of a pass (every ID twice)."""
    def whole(lo, hi):
        return torch.randint(lo, hi, (tasks * ids,), generator=gen, device=DEV, dtype=torch.int32)

    tuples = torch.ones((tasks * ids, 8), dtype=torch.int32, device=DEV)
    tuples[:, 0] = whole(0, 1 << 20)
    tuples[:, 1] = whole(1, 65536)
    tuples[:, 2] = 1 << whole(0, 7)
    tuples[:, 4] = 32 << whole(0, 6)
    tuples[:, 7] = 256 * whole(0, 257) * whole(0, 2)
    rho_e, rho_g = 0.95, 0.90          # share of the spread that belongs to the ID
    typical_e = LN(exec_ns) + rho_e * exec_sigma * torch.randn(tasks * ids, generator=gen, device=DEV)
    typical_g = LN(gap_ns) + rho_g * gap_sigma * torch.randn(tasks * ids, generator=gen, device=DEV)
    order = torch.rand((tasks, 2 * ids), generator=gen, device=DEV).argsort(dim=1) % ids
    return tuples, typical_e, typical_g, order


def _group_records(case, gen, out, lengths, ids, exec_ns, exec_sigma, gap_ns, gap_sigma, characters):
    """Writes the records of a group of tasks to out ([n, 64] bytes)."""
    words, quads = out.view(torch.int32), out.view(torch.int64)
    tuples, typical_e, typical_g, order = characters
    spread_e, spread_g = exec_sigma * math.sqrt(1 - 0.95 ** 2), gap_sigma * math.sqrt(1 - 0.90 ** 2)
    offsets = _offsets(lengths)
    cdf = None
    if case["pattern"] == "zipf":
        w = 1.0 / np.arange(1, ids + 1) ** 1.2
        cdf = torch.tensor(np.cumsum(w / w.sum()), dtype=torch.float32, device=DEV)
    first = 0
    while first < lengths.size:
        last = max(first + 1, int(np.searchsorted(offsets, offsets[first] + CHUNK, side="right")) - 1)
        a, b = int(offsets[first]), int(offsets[last])
        n = b - a
        lens = torch.from_numpy(lengths[first:last]).to(DEV)
        starts = torch.from_numpy(offsets[first:last] - a).to(DEV)
        task = torch.repeat_interleave(torch.arange(first, last, device=DEV), lens, output_size=n)
        at = torch.arange(n, device=DEV) - starts[task - first]
        if case["pattern"] == "pass":
            which = order[task, at % (2 * ids)]
        elif case["pattern"] == "uniform":
            which = torch.randint(0, ids, (n,), generator=gen, device=DEV)
        else:
            which = torch.searchsorted(cdf, torch.rand(n, generator=gen, device=DEV)).clamp_(max=ids - 1)
        which = task * ids + which
        words[a:b, :8] = tuples[which]
        e = torch.exp(typical_e[which] + spread_e * torch.randn(n, generator=gen, device=DEV)).round_().clamp_(min=1, max=4e9)
        g = torch.exp(typical_g[which] + spread_g * torch.randn(n, generator=gen, device=DEV)).round_()
        if case["stalls"]:
            stall = torch.exp(LN(200000.0) + 0.5 * torch.randn(n, generator=gen, device=DEV)).round_()
            g = torch.where(torch.rand(n, generator=gen, device=DEV) < case["stalls"], stall, g)
        if case["zero_gaps"]:
            g = torch.where(torch.rand(n, generator=gen, device=DEV) < case["zero_gaps"], torch.zeros_like(g), g)
        e, g = e.to(torch.int64), g.clamp_(max=4e9).to(torch.int64)
        end_of_gap = torch.cumsum(e + g, 0)
        begin = end_of_gap - e - g
        begin = begin - begin[starts[task - first]]
        quads[a:b, 4] = begin
        quads[a:b, 5] = begin + e
        quads[a:b, 6:8] = 0
        if case["runs"] > 1:
            words[a:b, 12] = (at * case["runs"] // lens[task - first]).to(torch.int32)
        first = last


def _records(case, gen, group_characters):
    hp, lp = _groups(case)
    out = torch.empty((int(hp.sum() + lp.sum()), 64), dtype=torch.uint8, device=DEV)
    n_hp = int(hp.sum())
    for which, lengths, part in (("hp", hp, out[:n_hp]), ("lp", lp, out[n_hp:])):
        if lengths.size:
            _group_records(case, gen, part, lengths, case[which + "_ids"], case[which + "_exec_ns"], case[which + "_exec_sigma"],
                           case[which + "_gap_ns"], case[which + "_gap_sigma"], group_characters[which])
    return out


def _both_characters(case, gen):
    got = {}
    for which in ("hp", "lp"):
        if case[which + "_tasks"]:
            got[which] = _characters(gen, case[which + "_tasks"], case[which + "_ids"], case[which + "_exec_ns"],
                                     case[which + "_exec_sigma"], case[which + "_gap_ns"], case[which + "_gap_sigma"])
    return got


def _empty(n, dtype=torch.int64):
    return torch.empty(n, dtype=dtype, device=DEV)


def _no_rows(capacity):
    """Space for rows, all zero: how many of them a call fills is up to the inputs, the rest is compared too."""
    return torch.zeros((capacity, 128), dtype=torch.uint8, device=DEV)


def _device(a, dtype=np.int64):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to(DEV)


def prepare(case, seed):
    """Records, offsets and scenarios on the GPU, and the output and work buffers that a program keeps from call to call."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    path = case["path"]
    hp_len, lp_len = _groups(case)
    off = _offsets(np.concatenate([hp_len, lp_len]))
    n, tasks = int(off[-1]), off.size - 1
    characters = _both_characters(case, gen)
    records = _records(case, gen, characters)
    d_off = _device(off)
    rows = _row_bound(case)
    s = {"case": case, "d_off": d_off, "n": n}
    hp, lp, gaps = _scenarios(case)
    n_gaps, n_scen = int(gaps[-1]), case["scenarios"]
    s.update(d_hp=_device(hp, np.int32), d_lp=_device(lp, np.int32), d_gaps=_device(gaps), n_gaps=n_gaps, tasks=tasks,
             predict=binding.FIKIT_PREDICT_MEAN if case["mean"] else binding.FIKIT_PREDICT_P50)

    def fill_out():
        return binding.GapFill(_empty(n_gaps, torch.int32), _empty(n_gaps), _empty(n_scen), _empty(n_scen))

    if path == "measure":
        s.update(records=records, exec_out=_empty(n), gap_out=_empty(n), ws=binding.workspace(256, DEV))
        return s
    if path in ("profile", "step"):
        nbytes = (binding.fikit_profile_workspace_bytes(n, tasks) if path == "profile"
                  else binding.fikit_profile_gapfill_workspace_bytes(n, tasks, n_scen))
        s.update(records=records, ids=_empty(n) if case["want_ids"] else None, rows=_no_rows(rows),
                 row_off=_empty(tasks + 1), ws=binding.workspace(nbytes, DEV))
        if path == "step":
            s.update(out=fill_out())
        return s

    # what the other calls start from is a profile of the same traces
    profile = binding.fikit_profile(records, d_off, row_capacity=rows)
    if path == "merge":
        # the further run: the same services, but a part of the tasks calls a different set of kernels now
        changed = torch.rand(tasks, generator=gen, device=DEV) < 0.25
        for tuples, _, _, _ in characters.values():
            ids = tuples.shape[0] // tasks
            tuples.view(tasks, ids, 8)[:, :ids // 4, 0] += changed.to(torch.int32)[:, None] << 20
        further = binding.fikit_profile(_records(case, gen, characters), d_off, row_capacity=rows)
        s.update(a=profile, b=further, rows=_no_rows(2 * rows), row_off=_empty(tasks + 1),
                 ws=binding.workspace(binding.fikit_profile_merge_workspace_bytes(tasks), DEV))
        return s
    s.update(profile=profile, out=fill_out())
    if path == "static":
        s.update(status=_empty(1, torch.int32))
    elif path == "gapfill":
        s.update(ws=binding.workspace(binding.fikit_gapfill_workspace_bytes(n, tasks, n_scen), DEV))
    elif path == "replay":
        o = s["out"]
        s.update(actual=binding.fikit_measure(records, d_off)[1],
                 out=binding.Replay(o.fill_count, o.filled_ns, o.lp_completion_ns, o.lp_placed),
                 ws=binding.workspace(binding.fikit_replay_workspace_bytes(n, tasks, n_scen), DEV))
    elif path == "prio":
        k = case["lists"]
        entry = np.arange(n_scen * k, dtype=np.int64)
        lists = case["hp_tasks"] + (lp[entry // k] - case["hp_tasks"] + entry % k) % case["lp_tasks"]
        levels = 1 + (entry // k // 3 + 2 * (entry % k // 2)) % 9      # neighbours in a list often share a level
        o = s["out"]
        s.update(d_lists=_device(lists, np.int32), d_levels=_device(levels, np.int32),
                 d_list_off=_device(np.arange(n_scen + 1, dtype=np.int64) * k),
                 out=binding.PrioFill(o.fill_count, o.filled_ns, _empty(n_scen * k), _empty(n_scen * k)),
                 ws=binding.workspace(binding.fikit_prio_fill_workspace_bytes(n, tasks, n_scen), DEV))
    elif path == "pairing":
        s["filled"] = binding.fikit_gapfill(profile.ids, d_off, profile.rows, profile.task_row_offsets, s["d_hp"], s["d_lp"], s["d_gaps"],
                                            margin_ns=500, min_gap_ns=case["min_gap_ns"], predictor=s["predict"], n_gaps=n_gaps,
                                            out=s["out"])
        s.update(out=binding.Pairing(_empty(n_scen), _empty(tasks), _empty(tasks, torch.int32), _empty(tasks)),
                 ws=binding.workspace(binding.fikit_pairing_workspace_bytes(tasks), DEV))
    return s


def run(s):
    """One call of the case's entry point and its outputs (rows together with the space behind them: their number depends on the
    inputs)."""
    case, path = s["case"], s["case"]["path"]
    if path == "step":
        profile, out = binding.fikit_profile_gapfill(
            s["records"], s["d_off"], s["d_hp"], s["d_lp"], s["d_gaps"], margin_ns=500, min_gap_ns=case["min_gap_ns"],
            predictor=s["predict"], n_gaps=s["n_gaps"], ids_out=s["ids"], rows_out=s["rows"], task_row_offsets_out=s["row_off"],
            out=s["out"], workspace_buf=s["ws"])
        return profile.ids, s["rows"], profile.task_row_offsets, profile.n_rows, out
    if path == "profile":
        profile = binding.fikit_profile(s["records"], s["d_off"], ids_out=s["ids"], rows_out=s["rows"], task_row_offsets_out=s["row_off"],
                                        workspace_buf=s["ws"], want_ids=case["want_ids"])
        return profile.ids, s["rows"], profile.task_row_offsets, profile.n_rows
    if path == "measure":
        return binding.fikit_measure(s["records"], s["d_off"], exec_out=s["exec_out"], gap_out=s["gap_out"], workspace_buf=s["ws"])
    if path == "merge":
        a, b = s["a"], s["b"]
        merged = binding.fikit_profile_merge(a.rows, a.task_row_offsets, b.rows, b.task_row_offsets, rows_out=s["rows"],
                                             task_row_offsets_out=s["row_off"], workspace_buf=s["ws"])
        return s["rows"], merged.task_row_offsets, merged.n_rows
    if path == "pairing":
        f = s["filled"]
        return binding.fikit_pairing_best(s["d_hp"], s["d_lp"], s["tasks"], s["d_gaps"], f.filled_ns, f.lp_completion_ns, out=s["out"],
                                          workspace_buf=s["ws"])
    p = s["profile"]
    common = dict(margin_ns=500, min_gap_ns=case["min_gap_ns"], predictor=s["predict"], n_gaps=s["n_gaps"], n_ids=s["n"], out=s["out"])
    if path == "static":
        binding.fikit_gapfill_static(p.ids, s["d_off"], p.rows, p.task_row_offsets, s["d_hp"], s["d_lp"], s["d_gaps"],
                                     status_out=s["status"], **common)
        return s["out"], s["status"]
    if path == "gapfill":
        return binding.fikit_gapfill(p.ids, s["d_off"], p.rows, p.task_row_offsets, s["d_hp"], s["d_lp"], s["d_gaps"],
                                     workspace_buf=s["ws"], **common)
    if path == "replay":
        return binding.fikit_gapfill_replay(p.ids, s["d_off"], p.rows, p.task_row_offsets, s["actual"], s["d_hp"], s["d_lp"],
                                            s["d_gaps"], feedback=case["feedback"], workspace_buf=s["ws"], **common)
    assert path == "prio", path
    return binding.fikit_prio_fill(p.ids, s["d_off"], p.rows, p.task_row_offsets, s["d_hp"], s["d_list_off"], s["d_lists"],
                                   s["d_levels"], s["d_gaps"], workspace_buf=s["ws"], **common)
