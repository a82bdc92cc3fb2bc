"""Who waits for whom when calls on several streams launch strips, two workgroups to a compute unit, and kernels whose
workgroups take a whole one: a model of one XCD as in test_strip_admission_cpu.py.  Only what may wait for ever is in it:
the workgroups that do the images of slots given up and the clusters' slots (up to 8 on an XCD of each).  A workgroup
takes one range of a compute unit's registers, and an adversary places what is pending, in any order, on any compute unit
and, with other kernels' waves beside it that have gone since, anywhere in a gap that holds it; whatever has all
its workgroups there ends."""
import os
import random
import re

import pytest

from tests.test_strip_admission_cpu import CSRC, MAX_GROUPS, QUEUES, REGISTERS, STRIP, UNITS, XCDS, gaps

WHOLE = REGISTERS
LEFT = (MAX_GROUPS // XCDS, WHOLE)                     # on an XCD, of a call
CLUSTERS = [(8, WHOLE), (8, REGISTERS // 2)]


def ends(kinds, rng):
    """`kinds`: per call the workgroups it needs there together and the registers (of 512 a SIMD) each takes."""
    taken = [[] for _ in range(UNITS)]                 # (base, size, call)
    there = [0] * len(kinds)
    done = [False] * len(kinds)
    while not all(done):
        moves = [(c, u) for c, (need, size) in enumerate(kinds) if not done[c] and there[c] < need
                 for u in range(UNITS) if gaps(taken[u], size)]
        if not moves:
            return False
        # the call that has most of its workgroups goes last, and fresh compute units are taken first
        few = min(there[c] - kinds[c][0] for c, _ in moves) if rng.random() < 0.5 else None
        c, u = rng.choice([m for m in moves if few is None or there[m[0]] - kinds[m[0]][0] == few])
        if rng.random() < 0.8:
            u = min((v for d, v in moves if d == c), key=lambda v: (len(taken[v]), rng.random()))
        low, high = rng.choice(gaps(taken[u], kinds[c][1]))
        taken[u].append((rng.randrange(low, high - kinds[c][1] + 1, 8), kinds[c][1], c))
        there[c] += 1
        if there[c] == kinds[c][0]:
            taken = [[t for t in unit if t[2] != c] for unit in taken]
            done[c] = True
    return True


def test_the_launch_is_the_models():
    """A workgroup per compute unit of a slot (at most kStripMaxGroups of them, dealt to the XCDs in turn), each of as
    many waves as fill its registers."""
    host = open(os.path.join(CSRC, "rtprune.hip")).read()
    device = open(os.path.join(CSRC, "sinkhorn_strip.hpp")).read()
    assert re.search(r"k_sinkhorn_strips_left<S>, dim3\(groups\), dim3\(kStripTeams \* kStripThreads\)", host)
    assert re.search(r"__launch_bounds__\(kStripTeams \* kStripThreads\) __attribute__\(\(amdgpu_waves_per_eu\(2, 2\)\)\) void "
                     r"k_sinkhorn_strips_left", device)
    assert re.search(r"kStripThreads = 256,.*kStripTeams = 2;", device)


@pytest.mark.parametrize("cluster", CLUSTERS)
@pytest.mark.parametrize("clusters", range(QUEUES + 1))
def test_those_that_wait_for_each_other_always_end(clusters, cluster):
    for seed in range(150):
        assert ends([cluster] * clusters + [LEFT] * (QUEUES - clusters), random.Random(seed)), (clusters, seed)


def test_twice_as_many_of_half_the_size_would_not():
    """(A compute unit that two of them fit on is no two places: one of them may lie in its middle.)"""
    half = (2 * MAX_GROUPS // XCDS, STRIP)
    assert not all(ends([half] * 3, random.Random(s)) for s in range(150))
