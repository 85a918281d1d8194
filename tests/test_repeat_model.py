"""The inputs of test_gpu_repeats.py take every way through the search for repeats and through the copy (followed on the host)."""
from collections import Counter

import numpy as np
import pytest

import oracle
from paper_2311_10359_amd import traces
from repeat_model import LIMITS, follow
from test_gpu_repeats import grid, stops, tasks_of


def happens(inputs, team, margins=((0, 0), (50, 500))):
    """What happens over the scenarios of all inputs; `wide`: copies of gaps that take something where the sums of a window pass 32 bits."""
    seen = Counter()
    for kids, exec_of, gap_of, h, l in inputs:
        rec, off = tasks_of(np.random.default_rng(1), kids, exec_of, gap_of)
        o_ids, o_rows, o_tro = oracle.profile(rec, off)
        gaps = traces.gap_offsets(off, h)
        pairs = {(a, b): s for s, (a, b) in enumerate(zip(h.tolist(), l.tolist()))}
        for margin, min_gap in margins:
            counts = oracle.gapfill(o_ids, off, o_rows, o_tro, h, l, margin, min_gap, gaps)[0]
            for (a, b), s in pairs.items():
                one = follow(gap_of[kids[a]], exec_of[kids[b]], counts[int(gaps[s]):int(gaps[s + 1])], team)[0]
                one["wide"] = one["copied_entries"] if int(exec_of.max()) >= 1 << 30 else 0
                seen += one
    return seen


WAYS = ("short_period", "false_start", "no_period", "doubled", "match_after_doubling", "all_notes", "queue_ends", "queue_short", "gave_up",
        "whole", "cut_by_gap", "cut_by_entry", "entry_behind_unit", "entry_last_of_unit", "cut_by_gap_and_entry", "nothing_held_gap",
        "nothing_held_entry", "again", "to_the_end", "last_unit_part", "copied_entries")


@pytest.mark.parametrize("team", [True, False])
def test_the_inputs_take_every_way(team):
    seen = {times: happens([grid(times, team)], team) for times in ("few", "many", "stuck", "zeros", "wide_sums")}
    seen["stops"] = happens([stops(team)], team)
    total = sum(seen.values(), Counter())
    assert not [way for way in WAYS + ("still" if team else "not_worth",) if not total[way]], total
    # gaps that take something are copied with kernels of no duration, and with windows whose sums do not fit 32 bits
    assert seen["zeros"]["copied_entries"] and seen["wide_sums"]["wide"], seen


def test_the_limits_are_read_from_the_source():
    assert {"GF_TEAM_SCENARIOS", "GF_TEAM_LAUNCHES", "GF_REPEAT_LAUNCHES", "REPEAT_GAPS", "REPEAT_ENTRIES", "REPEAT_WORTH", "REPEAT_LEAST", "REPEAT_NOTES",
            "REPEAT_MISSES", "REPEAT_ANCHOR", "REPEAT_ANCHORS"} <= set(LIMITS)
