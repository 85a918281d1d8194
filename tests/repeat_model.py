"""What the walk by wave copies, followed on the host: the search for repeats and the comparison, gap positions and all, on the predicted
times of one scenario and the entries that the oracle says its gaps took.  It tells which ways through the device code a test's inputs
take; whether results are right is for the oracle.  The limits are read from the kernels' source, so that both stay in step."""
import os
import re
from collections import Counter

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_10359_amd", "csrc")


def limits():
    """REPEAT_* and GF_* limits of the walk by their names in the source."""
    got = {}
    for name in ("gapfill_kernels.hip.h", "fikit.hip"):
        for line in open(os.path.join(CSRC, name)):
            m = re.match(r"constexpr (?:uint32_t|uint64_t|int) (.*?);", line)
            for key, value in re.findall(r"(\w+) = ([^,;]+)", m.group(1)) if m else ():
                if key.startswith(("REPEAT_", "GF_TEAM_", "GF_REPEAT_")):
                    got[key] = int(eval(value.replace("/", "//"), {}, got))
    return got


LIMITS = limits()
ROUND, BLOCK = 256, 64


def follow(G, q, counts, team):
    """G: idle time after each launch of the trace, q: the queue's durations, counts: entries that each gap took.  Returns a Counter of
    what happens, with the number of `copied` gaps, and the first repeat that is compared: gap, entry, gaps and entries of a unit."""
    seen, repeat = Counter(), None
    n_gaps, L = len(counts), len(q)
    J = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)      # where the queue stands before each gap
    gaps, q = G[:n_gaps], np.asarray(q)
    until = n_gaps - ROUND if n_gaps >= LIMITS["REPEAT_GAPS"] and L >= LIMITS["REPEAT_ENTRIES"] else 0

    def next_entries(j):
        return q[np.minimum(np.arange(j, j + BLOCK), L - 1)]

    i0 = misses = period = place = 0
    anchor, tries, next_anchor, notes = 0, 0, 0, []
    while i0 < until and J[i0] < L:
        first, start = i0, None
        if not period:
            if first >= next_anchor:
                anchor, tries = first, tries + 1
                if tries > LIMITS["REPEAT_ANCHORS"]:
                    seen["no_period"] += 1
                    break
                next_anchor = first + LIMITS["REPEAT_ANCHOR"] * (1 if tries < LIMITS["REPEAT_ANCHORS"] else 2)
            x = np.arange(first, first + ROUND)
            hit = (G[x] == G[anchor]) & (G[x + 1] == G[anchor + 1]) & ((x - first) % BLOCK != BLOCK - 1) & (x != anchor)
            if hit.any():
                start = int(x[hit][0])
        i0 = first + ROUND
        if J[i0] >= L:
            break                                                       # (the queue has been used up)
        if start is not None:
            if start + BLOCK <= len(G) and np.array_equal(G[anchor:anchor + BLOCK], G[start:start + BLOCK]):
                period = start - anchor
                if period < LIMITS["REPEAT_LEAST"]:
                    period *= -(-LIMITS["REPEAT_LEAST"] // period)
                    seen["short_period"] += 1
                place, notes = anchor + period, [(anchor, int(J[anchor]))]
            else:
                seen["false_start"] += 1
                misses += 1
                if misses >= LIMITS["REPEAT_MISSES"]:
                    until = 0
        if not period or place > i0:
            continue
        while place + period <= i0:
            place += period
        ja = int(J[place])
        match = [n for n in notes if np.array_equal(next_entries(n[1]), next_entries(ja))]
        units = 0
        if match:
            a, (from_i, from_j) = place, match[-1]
            D, dq = a - from_i, ja - from_j
            wanted = -(-(n_gaps - a) // D)
            there = (L - 1 - ja) // dq if dq else wanted
            units = min(wanted, there)
            X = n_gaps if units == wanted else a + units * D
            if X <= i0:
                units = 0
            if there == 0:
                seen["queue_ends"] += 1
                until = 0
            if not team and dq < D // LIMITS["REPEAT_WORTH"]:
                seen["not_worth"] += 1
                units = until = 0
            if units:
                seen["match_after_doubling"] += len(notes) >= 16
        notes.append((place, ja))
        if len(notes) % 16 == 0:
            seen["doubled"] += 1
            period *= 2
        if len(notes) >= LIMITS["REPEAT_NOTES"]:
            seen["all_notes"] += 1
            until = 0
        place += period
        if not units:
            continue
        # what is compared
        repeat = repeat or (a, ja, D, dq)
        at = np.arange(a, X)
        bad = np.flatnonzero(gaps[at] != gaps[a - D + (at - a) % D])
        bad_x = int(at[bad[0]]) if bad.size else None
        hold, cut = units, None
        if bad_x is not None:
            hold, cut = (bad_x - a) // D, "gap"
        if dq and a + hold * D > i0:
            last = ja + hold * dq
            y = np.arange(ja, last + 1)
            bad = np.flatnonzero(q[y] != q[y - dq])
            if bad.size:
                bad_y = int(y[bad[0]])
                n = (bad_y - ja - 1) // dq if bad_y > ja else 0
                if n < hold:
                    seen["cut_by_gap_and_entry"] += cut == "gap"
                    hold, cut = n, "entry"
                    if a + hold * D > i0:
                        seen["entry_behind_unit"] += (bad_y - ja) % dq == 0
                        seen["entry_last_of_unit"] += (bad_y - ja) % dq == dq - 1
        end = n_gaps if hold == wanted else a + hold * D
        copied = max(0, end - i0)
        if copied:
            seen["copies"] += 1
            seen["copied"] += copied
            seen["copied_entries"] += int(J[end] - J[i0])
            seen["still"] += dq == 0
            seen["cut_by_" + cut if cut else "whole"] += 1
            seen["again"] += seen["copies"] > 1
            seen["to_the_end"] += end == n_gaps
            seen["last_unit_part"] += end == n_gaps and (n_gaps - a) % D != 0
            seen["queue_short"] += cut is None and end < n_gaps
        else:
            seen["nothing_held_" + (cut or "")] += 1
        if cut:
            misses = misses + 2 if copied < LIMITS["REPEAT_ANCHOR"] else 0
            if misses >= LIMITS["REPEAT_MISSES"]:
                until = 0
                seen["gave_up"] += 1
            period, anchor, tries, next_anchor = 0, 0, 0, 0
        if copied:
            i0 = end
            if period:
                place = end + period
    return seen, repeat
