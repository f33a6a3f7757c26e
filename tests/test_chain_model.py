"""CPU model of the chain scan's tiles and their look-back (no GPU).

In the scan (paper_2406_10158_amd/csrc/chain.hip) a workgroup takes the next
tile of the accesses sorted by cell, loads the initial value of every chain
that begins in it, publishes its state, looks back for the value on entry if
its first access continues a chain, and stores the cell of every chain that
ends in it.  The workgroups of a launch run at the same time, so a chain's
first tile may still have its load in flight when another tile stores the
chain's final value into the same word.

The model steps the running tiles in random order, with the load a step that
completes at any later time, and replays the batch in order for comparison.
It has both rules: the kernel's (a tile publishes once its loads are complete,
and one that ends a chain it did not begin stores the cell only once it has
seen a settled tile), and the rule without the two waits, under which the
first tile can load the final value -- so that the model is known to see the
fault.
"""
from __future__ import annotations

import random

import pytest

REL, ABS, BRK = range(3)


def then(x, y):
    return y if y[0] != REL else (x[0], x[1] + y[1])


def effect(op):
    return {"add": (REL, op[1]), "const": (ABS, op[1]), "brk": (BRK, 0)}[op[0]]


class Scan:
    """accesses: (cell, op) sorted by cell; a break's result is taken as relative to nothing (BRK, sums after it)."""

    def __init__(self, accesses, cells, tile, running, rng, ordered):
        self.acc, self.data, self.tile, self.rng, self.ordered = accesses, list(cells), tile, rng, ordered
        self.n_tiles = -(-len(accesses) // tile)
        self.meta = [None] * self.n_tiles  # (total known, value, settled)
        self.read = [None] * len(accesses)
        self.queue = 0
        self.slots = [None] * running

    def run(self):
        speed = [self.rng.choice([1, 100]) for _ in self.slots]  # a slow workgroup is far behind the others
        for _ in range(100_000):
            i = self.rng.choices(range(len(self.slots)), speed)[0]
            if self.slots[i] is None and self.queue < self.n_tiles:
                self.slots[i] = self.workgroup(self.queue)
                self.queue += 1
            if self.slots[i] is not None and next(self.slots[i], "end") == "end":
                self.slots[i] = None
            if self.queue == self.n_tiles and not any(self.slots):
                return
        raise AssertionError("a tile waits forever")

    def workgroup(self, t):
        p0, p1 = t * self.tile, min((t + 1) * self.tile, len(self.acc))
        cell = [c for c, _ in self.acc[p0:p1]]
        head = [p == 0 or self.acc[p - 1][0] != self.acc[p][0] for p in range(p0, p1)]
        last = [p + 1 == len(self.acc) or self.acc[p + 1][0] != self.acc[p][0] for p in range(p0, p1)]
        init = {}
        waiting = [i for i, h in enumerate(head) if h]

        def total():
            run = (REL, 0)
            for i, (_, op) in enumerate(self.acc[p0:p1]):
                if head[i]:
                    run = (ABS, init.get(i, 0))
                run = then(run, effect(op))
            return run

        def load():
            i = waiting.pop(self.rng.randrange(len(waiting)))
            init[i] = self.data[cell[i]]

        # what is published needs the loads it is computed from; the others may still be in flight
        while waiting and (self.ordered or self.needed(p0, p1, head) & set(waiting)):
            yield
            load()
        yield
        all_ = total()
        self.meta[t] = (all_[0] != REL, all_, any(head))
        entry, settled = (REL, 0), True
        if not head[0]:
            at, entry = t - 1, (REL, 0)
            while True:
                yield
                if self.meta[at] is None:
                    continue
                known, v, settled = self.meta[at]
                entry = then(v, entry)
                if known:
                    break
                at -= 1
            if all_[0] == REL:
                yield
                self.meta[t] = (True, then(entry, all_), settled)
            at = t - 1
            while self.ordered and any(last) and not settled:
                yield
                if self.meta[at] is None:
                    continue
                settled = self.meta[at][2]
                at -= 1
        st = entry
        for i, (c, op) in enumerate(self.acc[p0:p1]):
            if head[i]:
                while i in waiting:
                    yield
                    load()
                st = (ABS, init[i])
            self.read[p0 + i] = st
            st = then(st, effect(op))
            if last[i] and st[0] == ABS:
                yield
                self.data[c] = st[1]

    def needed(self, p0, p1, head):
        """Chain heads whose initial value the tile's total depends on."""
        need = set()
        for i, (_, op) in enumerate(self.acc[p0:p1]):
            if head[i]:
                need = {i}
            if effect(op)[0] != REL:
                need = set()
        return need


def expected(accesses, cells):
    data, read, at = list(cells), [], None
    st = (REL, 0)
    for p, (c, op) in enumerate(accesses):
        if c != at:
            at, st = c, (ABS, data[c])
        read.append(st)
        st = then(st, effect(op))
        if (p + 1 == len(accesses) or accesses[p + 1][0] != c) and st[0] == ABS:
            data[c] = st[1]
    return read, data


def chains(rng, lengths, consts, breaks):
    """A chain per cell: adds, with a constant or a break at a share of the places."""
    acc = []
    for c, n in enumerate(lengths):
        for _ in range(n):
            r = rng.random()
            kind = "const" if r < consts else ("brk" if r < consts + breaks else "add")
            acc.append((c, (kind, rng.randint(1, 9))))
    return acc


def wrong(ordered, lengths, consts, breaks, seeds=400):
    bad = 0
    for seed in range(seeds):
        rng = random.Random(seed)
        acc = chains(rng, lengths, consts, breaks)
        cells = [1000 * (i + 1) for i in range(len(lengths))]
        s = Scan(acc, cells, 4, 7, rng, ordered)
        s.run()
        bad += (s.read, s.data) != expected(acc, cells)
    return bad


CASES = [
    ([30], 0.2, 0.0),           # one cell over eight tiles, constants here and there
    ([30], 0.3, 0.0),
    ([2, 27, 3], 0.2, 0.0),     # its first and last tiles shared with other cells
    ([30], 0.2, 0.1),           # breaks too: a total that is known without the entry either
    ([5, 9, 13, 17], 0.15, 0.1),
    ([40], 0.0, 0.0),           # adds alone
]


@pytest.mark.parametrize("lengths,consts,breaks", CASES)
def test_every_interleaving_gives_the_replays_values(lengths, consts, breaks):
    assert wrong(True, lengths, consts, breaks) == 0


@pytest.mark.parametrize("lengths,consts,breaks", CASES[:4])
def test_without_the_waits_a_chains_first_tile_loads_its_last_value(lengths, consts, breaks):
    assert wrong(False, lengths, consts, breaks) > 0
