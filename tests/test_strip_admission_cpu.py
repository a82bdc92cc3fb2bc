"""Who waits for whom when calls on several streams launch strips at once, as a model: eight XCDs of 32 compute
units, a launch's workgroups dealt to the XCDs in turn and placed on each in order, one to a compute unit, by an
adversary who chooses which launch gets the next free place, when a wait runs out and when a slot ends.  The
constants are the kernels' own (csrc/sinkhorn_team.hpp)."""
import os
import random
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_00392_amd", "csrc")
TEAM = open(os.path.join(CSRC, "sinkhorn_team.hpp")).read()


def constant(name):
    return int(re.search(rf"\b{name} = (\d+)", TEAM).group(1))


XCDS, UNITS, QUEUES = 8, 32, 4
XCD_GROUPS, MAX_GROUPS, MAX_SLOTS = constant("kStripXcdGroups"), constant("kStripMaxGroups"), constant("kStripMaxSlots")


class Launch:
    """Slots of `groups` workgroups, as many as the chip holds, and, with `last`, the last workgroups."""

    def __init__(self, groups, last):
        cus = XCDS * UNITS
        self.groups, self.has_last = groups, last
        self.local = groups <= XCD_GROUPS
        self.slots = 8 * min(MAX_SLOTS // 8, cus // 8 // groups) if self.local else min(MAX_SLOTS, cus // groups)
        blocks = [self.slot_of(b) for b in range(self.slots * groups)] + ["last"] * (groups if last else 0)
        self.pending = [[blocks[b] for b in range(x, len(blocks), XCDS)] for x in range(XCDS)]
        self.there = {}                                # slot -> workgroups of it that are resident
        self.state = {}                                # slot -> "complete" / "given up" / "done"

    def slot_of(self, b):
        return (b % 8) * (self.slots // 8) + b // 8 // self.groups if self.local else b // self.groups

    def settled(self):
        return all(self.state.get(s) for s in range(self.slots))


def run(launches, rng):
    """True when everything ends."""
    used = [[] for _ in range(XCDS)]                   # (launch, slot) of every workgroup that holds a compute unit
    while True:
        moves = []
        for x in range(XCDS):
            if len(used[x]) < UNITS:
                moves += [("place", l, x) for l in launches if l.pending[x]]
        for l in launches:
            for s, n in l.there.items():
                if not n:
                    continue
                if s == "last":
                    # they leave when every slot is settled and none was given up, or when they have all met
                    if l.settled() and ("given up" not in l.state.values() or n == l.groups):
                        moves.append(("end", l, s))
                    elif not l.settled():
                        moves.append(("give up", l, next(t for t in range(l.slots) if not l.state.get(t))))
                elif l.state.get(s) in ("complete", "given up", "done"):
                    moves.append(("end", l, s))
                elif l.has_last:                       # a bounded wait
                    moves.append(("give up", l, s))
        if not moves:
            return not any(used) and not any(p for l in launches for p in l.pending)
        # the adversary: waits run out as late as possible
        early = [m for m in moves if m[0] == "place"] or [m for m in moves if m[0] == "end"] or moves
        kind, l, a = rng.choice(early if rng.random() < 0.97 else moves)
        if kind == "place":
            s = l.pending[a].pop(0)
            if l.state.get(s) == "given up":           # (it looks and leaves)
                continue
            used[a].append((l, s))
            l.there[s] = l.there.get(s, 0) + 1
            if s != "last" and l.there[s] == l.groups:
                l.state[s] = "complete"
        elif kind == "give up":
            l.state[a] = "given up"
        else:
            for x in range(XCDS):
                used[x] = [u for u in used[x] if u != (l, a)]
            l.there[a] = 0
            if a == "last" and "given up" in l.state.values():
                l.state.update({t: "done" for t, v in l.state.items() if v == "given up"})


MIXES = [(16, 16, 16), (9, 9, 9, 9), (16, 12, 14, 11), (58, 58), (64, 64, 64, 64), (24, 40, 16, 64), (17, 17, 17, 17),
         (4, 16, 58, 9), (8, 8, 8, 8)]


@pytest.mark.parametrize("mix", MIXES)
def test_up_to_four_calls_always_end(mix):
    assert len(mix) <= QUEUES and max(mix) <= MAX_GROUPS
    for seed in range(60):
        assert run([Launch(g, True) for g in mix], random.Random(seed)), (mix, seed)


def test_slots_that_wait_for_ever_would_not():
    stuck = [mix for mix in MIXES if not all(run([Launch(g, False) for g in mix], random.Random(s)) for s in range(60))]
    assert (16, 16, 16) in stuck and (9, 9, 9, 9) in stuck and (64, 64, 64, 64) in stuck, stuck
    assert (8, 8, 8, 8) not in stuck                   # up to eight workgroups on an XCD: 4 * 7 < 32
