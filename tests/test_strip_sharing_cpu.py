"""Who waits for whom when calls on several streams launch strips, two workgroups to a compute unit, and kernels whose
workgroups take a whole one: a model as in test_strip_admission_cpu.py.  Only what may wait for ever is in it:
a strip launch's last workgroups (up to 16 on an XCD, half a compute unit each) and the clusters' slots (up
to 8, a whole one each).  An adversary places what is pending, in any order and on either half of any compute
unit; whatever has all its workgroups there ends."""
import random

import pytest

from tests.test_strip_admission_cpu import MAX_GROUPS, QUEUES, UNITS, XCDS


def ends(kinds, rng):
    """One XCD; `kinds`: per call the workgroups it needs there together and the halves each takes."""
    free = [2] * UNITS
    there = [[] for _ in kinds]
    done = [False] * len(kinds)
    while not all(done):
        moves = [(c, u) for c, (need, size) in enumerate(kinds) if not done[c] and len(there[c]) < need
                 for u in range(UNITS) if free[u] >= size]
        if not moves:
            return False
        # the call that has most of its workgroups goes last, and fresh compute units are taken first
        few = min(len(there[c]) - kinds[c][0] for c, _ in moves) if rng.random() < 0.5 else None
        c, u = rng.choice([m for m in moves if few is None or len(there[m[0]]) - kinds[m[0]][0] == few])
        if rng.random() < 0.8:
            u = max((v for d, v in moves if d == c), key=lambda v: (free[v], rng.random()))
        there[c].append(u)
        free[u] -= kinds[c][1]
        if len(there[c]) == kinds[c][0]:
            for u in there[c]:
                free[u] += kinds[c][1]
            done[c] = True
    return True


@pytest.mark.parametrize("clusters", range(QUEUES + 1))
def test_halves_and_whole_compute_units_always_end(clusters):
    half = (2 * MAX_GROUPS // XCDS, 1)
    for seed in range(300):
        assert ends([(8, 2)] * clusters + [half] * (QUEUES - clusters), random.Random(seed)), (clusters, seed)


def test_more_workgroups_to_an_xcd_would_not():
    assert not all(ends([(22, 1)] * QUEUES, random.Random(s)) for s in range(300))
