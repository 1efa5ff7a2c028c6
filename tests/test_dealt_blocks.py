"""The block order that gives groups (slabs, windows, column groups) to the 8 XCDs,
csrc/bl_internal.h's dealt_blocks and dealt_task compiled for the host: every
(group, part) exactly once, whole rounds of groups on one XCD each, and the rest in
runs that differ by at most the rounding of one block per XCD; near the most blocks
that a launch takes, where 32-bit products could wrap, sampled blocks against the
same arithmetic in Python."""
import os
import subprocess

import pytest

XCDS = 8
HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("dealt") / "dealt_blocks")
    r = subprocess.run([os.path.join(ROCM, "llvm", "bin", "clang++"), "-O1", "-std=c++17",
                        "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                        os.path.join(HERE, "c", "dealt_blocks.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


def dealt(exe, groups, parts, first=0, step=1):
    """(blocks of the launch, [(block, group, part)]), group -1: no task."""
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    r = subprocess.run([exe], input=f"{groups} {parts} {first} {step}\n", capture_output=True,
                       text=True, env=env)
    assert r.returncode == 0, r.stderr
    head, *rows = r.stdout.splitlines()
    return int(head.split()[1]), [tuple(int(v) for v in row.split()) for row in rows]


@pytest.mark.parametrize("groups", [1, 2, 7, 8, 9, 15, 16, 98])
@pytest.mark.parametrize("parts", [1, 2, 3, 7, 8, 9, 125])
def test_every_block_once_and_evenly(exe, groups, parts):
    blocks, tasks = dealt(exe, groups, parts)
    assert len(tasks) == blocks
    seen = [(b % XCDS, g, p) for b, g, p in tasks if g >= 0]
    assert sorted((g, p) for _, g, p in seen) == [(g, p) for g in range(groups)
                                                  for p in range(parts)]
    assert all(x == g % XCDS for x, g, _ in seen if g < groups // XCDS * XCDS)
    load = [sum(1 for x, _, _ in seen if x == i) for i in range(XCDS)]
    assert max(load) <= groups // XCDS * parts + -(-(groups % XCDS * parts) // XCDS)


@pytest.mark.parametrize("groups,parts", [(7, 306783377), (1, 2147483640), (15, 143165576),
                                          (8, 268435455), (2147483640, 1), (2147483639, 1),
                                          (65535, 32767)])
def test_the_largest_launches(exe, groups, parts):
    rounds, rest = groups // XCDS, groups % XCDS * parts
    run = -(-rest // XCDS)
    blocks = XCDS * (rounds * parts + run)
    assert 0x7fffffff - 2 * 65536 < blocks <= 0x7fffffff
    for first, step in ((0, 50000017), (blocks - 40, 1)):
        n, tasks = dealt(exe, groups, parts, first, step)
        assert n == blocks and tasks
        for b, g, p in tasks:
            xcd, loc = b % XCDS, b // XCDS
            if loc < rounds * parts:
                want = (loc // parts * XCDS + xcd, loc % parts)
            else:
                e = xcd * run + loc - rounds * parts
                want = (rounds * XCDS + e // parts, e % parts) if e < rest else (-1, -1)
            assert (g, p) == want, (b, want)
