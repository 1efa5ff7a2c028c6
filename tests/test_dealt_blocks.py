"""The block order that gives groups (slabs, windows, column groups) to the 8
XCDs, in a model of csrc/bl_internal.h's dealt_blocks and dealt_task: every
(group, part) exactly once, whole rounds of groups on one XCD each, and the rest
in runs that differ by at most the rounding of one block per XCD."""
import pytest

XCDS = 8


def dealt(groups, parts):
    rounds, rest = groups // XCDS, groups % XCDS * parts
    run = (rest + XCDS - 1) // XCDS
    for bid in range(XCDS * (rounds * parts + run)):
        xcd, loc = bid % XCDS, bid // XCDS
        if loc < rounds * parts:
            yield xcd, loc // parts * XCDS + xcd, loc % parts
        else:
            e = xcd * run + loc - rounds * parts
            if e < rest:
                yield xcd, rounds * XCDS + e // parts, e % parts


@pytest.mark.parametrize("groups", [1, 2, 7, 8, 9, 15, 16, 98])
@pytest.mark.parametrize("parts", [1, 2, 3, 7, 8, 9, 125])
def test_every_block_once_and_evenly(groups, parts):
    seen = list(dealt(groups, parts))
    assert sorted((g, p) for _, g, p in seen) == [(g, p) for g in range(groups)
                                                  for p in range(parts)]
    assert all(x == g % XCDS for x, g, _ in seen if g < groups // XCDS * XCDS)
    load = [sum(1 for x, _, _ in seen if x == i) for i in range(XCDS)]
    assert max(load) <= groups // XCDS * parts + -(-(groups % XCDS * parts) // XCDS)
