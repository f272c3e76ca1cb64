"""The arrival counters of the small decode launches (csrc/eden_kernels_small.hip, k_dec_small), as a model on the CPU.

A launch of several workgroups counts arrivals in one word: the workgroup that brings it to the total adds the sums of all of
them and puts the word back to 0.  Two calls that overlap on one context are against the rules and get wrong sums; the model
runs random interleavings of two such launches and asks what the launches after them find."""
import os
import random
import re

import pytest

SOURCES = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2108_08842_amd", "csrc")


def _workgroup(words, turn, total, first, lasts):
    """One workgroup of a launch; yields between its accesses to memory."""
    if first:
        for i in range(len(words)):
            if i != turn:
                words[i] = 0
                yield
    words[turn] += 1                             # atomic
    arrived = words[turn]
    yield
    if arrived == total:
        lasts.append(arrived)
        words[turn] = 0
        yield


def _run(workgroups, order):
    for w in order:
        next(workgroups[w], None)
    for w in workgroups:                         # (a workgroup always finishes)
        for _ in w:
            pass


def _later_launches_are_right(counters, order, totals):
    words, turn, lasts = [0] * counters, 0, []
    overlapping = []
    for total in totals:
        overlapping += [_workgroup(words, turn, total, k == 0, lasts) for k in range(total)]
        turn = (turn + 1) % counters
    _run(overlapping, order)
    for total in (2, 3, 2, 2, 3) + (2,) * counters:              # from here on by the rules: one after the other
        lasts.clear()
        _run([_workgroup(words, turn, total, k == 0, lasts) for k in range(total)], ())
        if lasts != [total] or words[turn] != 0:
            return False
        turn = (turn + 1) % counters
    return True


@pytest.mark.parametrize("totals", [(2, 2), (2, 3), (3, 2)])
def test_launches_after_an_overlap_find_their_counter_at_zero(totals):
    source = open(os.path.join(SOURCES, "eden_device.h")).read()
    counters = int(re.search(r"kDecCounters = (\d+);", source).group(1))
    assert counters >= 3
    kernel = open(os.path.join(SOURCES, "eden_kernels_small.hip")).read()
    assert "threadIdx.x < kDecCounters && threadIdx.x != turn) arrived[threadIdx.x] = 0u;" in kernel
    # steps: the first workgroup of a launch clears two other words here, everyone counts, the last one resets.  (Three counters
    # show what any number from three on does: those of the launches that overlap, one that nothing has touched, and so on in turn.)
    first = [k in (0, totals[0]) for k in range(sum(totals))]
    steps = [w for w, f in enumerate(first) for _ in range(4 if f else 2)]
    rng = random.Random(7)
    orders = [rng.sample(steps, len(steps)) for _ in range(5000)]
    assert all(_later_launches_are_right(3, order, totals) for order in orders)
    assert not all(_later_launches_are_right(1, order, totals) for order in orders)      # one word, cleared by nobody else
