"""Who waits for whom when calls on several streams launch strips at once, as a model: eight XCDs of 32 compute
units, a launch's workgroups dealt to the XCDs in turn and placed on each in order, two to a compute unit where its
registers have a range left for the second, by an adversary who chooses which launch gets the next free place and where,
when other kernels' waves come and go, when a wait runs out and when a slot ends.  Behind a launch come the workgroups
that do the images of its slots given up, a whole compute unit each.  The constants are the kernels' own
(csrc/sinkhorn_team.hpp)."""
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
REGISTERS, STRIP = 512, 256                            # a SIMD's, and what a strip workgroup's wave there takes
OTHERS = (128, 156, 200, 230)                          # other kernels' waves


def gaps(taken, size):
    """The ranges between `taken` (base, size, ...) of a compute unit that hold `size` registers."""
    out, at = [], 0
    for base, held, *_ in sorted(taken) + [(REGISTERS, 0)]:
        if base - at >= size:
            out.append((at, base))
        at = base + held
    return out


class Unit:
    def __init__(self, taken):
        self.change(taken)

    def change(self, taken):
        self.taken = taken
        self.room = max((high - low for low, high in gaps(taken, 1)), default=0)


class Launch:
    """Slots of `groups` compute units, as many as the chip holds.  `bounded`: a slot that does not get complete is
    given up, and its images are done behind the launch."""

    def __init__(self, groups, bounded=True):
        cus = XCDS * UNITS
        self.groups, self.bounded, self.per_slot = groups, bounded, 2 * groups
        self.local = groups <= XCD_GROUPS
        self.slots = 8 * min(MAX_SLOTS // 8, cus // 8 // groups) if self.local else min(MAX_SLOTS, cus // groups)
        blocks = [self.slot_of(b) for b in range(self.slots * self.per_slot)]
        self.pending = [[blocks[b] for b in range(x, len(blocks), XCDS)] for x in range(XCDS)]
        self.there = {}                                # slot -> workgroups of it that are resident
        self.state = {}                                # slot -> "complete" / "given up" / "done"
        self.left = False                              # the second launch has been issued

    def slot_of(self, b):
        return (b % 8) * (self.slots // 8) + b // 8 // self.per_slot if self.local else b // self.per_slot

    def size(self, slot):
        return REGISTERS if slot == "left" else STRIP

    def next_launch(self):
        if not self.left and not any(self.pending) and not any(self.there.values()):
            self.left = True
            if "given up" in self.state.values():
                self.pending = [["left"] * len(range(x, self.groups, XCDS)) for x in range(XCDS)]


def run(launches, rng):
    """True when everything ends."""
    # (base, size, launch, slot) of every workgroup and (base, size, None, None) of other kernels' waves
    units = [[Unit([(0, rng.choice(OTHERS), None, None)] if rng.random() < 0.5 else []) for _ in range(UNITS)] for _ in range(XCDS)]

    def drop(which):
        for x in units:
            for u in x:
                if any(which(t) for t in u.taken):
                    u.change([t for t in u.taken if not which(t)])

    while True:
        for l in launches:
            l.next_launch()
        moves = [("place", l, x) for x in range(XCDS) for l in launches
                 if l.pending[x] and any(u.room >= l.size(l.pending[x][0]) for u in units[x])]
        if not moves or rng.random() < 0.02:
            if any(t[2] is None for x in units for u in x for t in u.taken):
                moves.append(("others end", None, None))
        for l in launches:
            for s, n in l.there.items():
                if not n:
                    continue
                if s == "left":
                    if n == l.groups:
                        moves.append(("end", l, s))
                elif l.state.get(s) in ("complete", "given up"):
                    moves.append(("end", l, s))
                elif l.bounded:                        # a bounded wait
                    moves.append(("give up", l, s))
        if not moves:
            return not any(u.taken for x in units for u in x) and not any(p for l in launches for p in l.pending)
        # the adversary: waits run out as late as possible
        early = [m for m in moves if m[0] == "place"] or [m for m in moves if m[0] != "give up"] or moves
        kind, l, a = rng.choice(early if rng.random() < 0.97 else moves)
        if kind == "place":
            s = l.pending[a].pop(0)
            if l.state.get(s) == "given up":           # (it looks and leaves)
                continue
            unit = rng.choice([u for u in units[a] if u.room >= l.size(s)])
            unit.change(unit.taken + [(rng.choice(gaps(unit.taken, l.size(s)))[0], l.size(s), l, s)])
            l.there[s] = l.there.get(s, 0) + 1
            if s != "left" and l.there[s] == l.per_slot:
                l.state[s] = "complete"
            if rng.random() < 0.3:                     # another kernel's wave comes
                size, unit = rng.choice(OTHERS), rng.choice(units[rng.randrange(XCDS)])
                if unit.room >= size:
                    unit.change(unit.taken + [(gaps(unit.taken, size)[0][0], size, None, None)])
        elif kind == "others end":
            drop(lambda t: t[2] is None and rng.random() < 0.7)
        elif kind == "give up":
            l.state[a] = "given up"
        else:
            drop(lambda t: t[2] is l and t[3] == a)
            l.there[a] = 0
            if a == "left":
                l.state.update({t: "done" for t, v in l.state.items() if v == "given up"})


MIXES = [(16, 16, 16), (9, 9, 9, 9), (16, 12, 14, 11), (58, 58), (64, 64, 64, 64), (24, 40, 16, 64), (17, 17, 17, 17),
         (4, 16, 58, 9), (8, 8, 8, 8)]


@pytest.mark.parametrize("mix", MIXES)
def test_up_to_four_calls_always_end(mix):
    assert len(mix) <= QUEUES and max(mix) <= MAX_GROUPS
    for seed in range(8):
        launches = [Launch(g) for g in mix]
        assert run(launches, random.Random(seed)), (mix, seed)
        assert all(l.state.get(s) in ("complete", "done") for l in launches for s in range(l.slots)), (mix, seed)


def test_slots_that_wait_for_ever_would_not():
    stuck = [mix for mix in MIXES if not all(run([Launch(g, False) for g in mix], random.Random(s)) for s in range(6))]
    assert (16, 16, 16) in stuck and (9, 9, 9, 9) in stuck and (64, 64, 64, 64) in stuck, stuck
