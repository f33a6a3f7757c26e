"""The chain scan (GaccO's and GPUTx's execution) where it can go wrong.

Single cells whose chains end around a tile of 2,048 accesses or span more
than the 64 tiles a look-back reads at once, made of adds, of conditional
adds (each a break the scan cannot see through) and of slot writes whose
source's own chain has breaks; operations that no transaction names, at the
end of a chain that a break is part of.  Every read value and cell is compared
with the oracle's id-order replay.
"""
import numpy as np
import pytest

import oracle
from helpers import binding
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu
TILE = 2048


def _batch(n_ops, row, field, kind, arg):
    n_ops = np.asarray(n_ops, np.uint32)
    first = (np.cumsum(n_ops) - n_ops).astype(np.uint64)
    return wl.Batch(first, n_ops, np.asarray(row, np.uint32), np.zeros(len(row), np.uint16),
                    np.asarray(field, np.uint8), np.asarray(kind, np.uint8), np.asarray(arg, np.int64))


def _check(tables, b, scheme, flags=0, gaps=0):
    b_ = binding()
    txns, ops = b_.pack_batch(b)
    ops = np.concatenate([ops, np.zeros(gaps, ops.dtype)])  # operations past the last transaction's
    print(f"[gpu] chain {scheme} ops={len(ops)} gaps={gaps}", flush=True)
    with b_.Engine(tables) as eng:
        bid = b_.cc_submit_batch(eng.ctx, txns, ops, b_.SCHEMES[scheme])
        eng.run(bid, flags=flags)
        out, reads = eng.outcomes(bid, b.n_txns, len(ops))
        final = eng.tables()
    exp_fin, exp_reads = oracle.id_order_expected(tables, b)
    assert np.all(out["status"] == oracle.COMMITTED)
    assert np.array_equal(reads[:b.total_ops], exp_reads)
    assert not reads[b.total_ops:].any()
    assert all(np.array_equal(g, e) for g, e in zip(final, exp_fin))


@pytest.mark.parametrize("scheme", ["gacco", "gputx"])
@pytest.mark.parametrize("kinds", [(wl.READ, wl.ADD), (wl.READ, wl.ADD, wl.COND_ADD), (wl.COND_ADD,)])
@pytest.mark.parametrize("n", [1, 63, 65, TILE - 1, TILE, TILE + 1, 3 * TILE + 5])
def test_chain_lengths_around_a_tile(n, kinds, scheme):
    # one cell's chain of n accesses between two short ones
    rng = np.random.default_rng(n)
    m = n + 5
    row = np.ones(m)
    row[[0, 1]] = 0
    row[[m - 2, m - 1, m - 3]] = 2
    b = _batch(np.ones(m), row, np.zeros(m), rng.choice(kinds, m), rng.integers(-30, 6, m))
    _check([wl.kv_table(3, 1)], b, scheme)


@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("breaks", [0, 0.0005])
def test_chain_longer_than_one_look_back(breaks, strict):
    # 70 tiles on one cell: look-backs cross the 64-tile window, to the chain's head or to a break
    rng = np.random.default_rng(7)
    m = 70 * TILE + 9
    kind = np.where(rng.random(m) < breaks, wl.COND_ADD, wl.ADD)
    b = _batch(np.ones(m), np.zeros(m), np.zeros(m), kind, rng.integers(-30, 31, m))
    _check([wl.kv_table(1, 1)], b, "gacco", flags=binding().CC_RUN_STRICT_FENCES if strict else 0)


@pytest.mark.parametrize("scheme", ["gacco", "gputx"])
@pytest.mark.parametrize("gaps", [0, 1, 100])
def test_slot_writes_follow_their_sources_breaks(gaps, scheme):
    # (read or conditional add on a hot cell, slot write elsewhere from its value): the slot's
    # cells feed further slots, constants (multiplier 0) among them; gaps end cell 0's chain
    rng = np.random.default_rng(11)
    n, rows = 3_000, 40
    row, kind, arg = np.zeros((n, 2)), np.zeros((n, 2)), np.zeros((n, 2), np.int64)
    row[:, 0] = rng.integers(0, 4, n) * (rng.random(n) < 0.9)
    row[:, 1] = rng.integers(4, rows, n)
    swap = rng.random(n) < 0.3
    row[swap] = row[swap][:, ::-1]
    kind[:, 0] = rng.choice([wl.READ, wl.ADD, wl.COND_ADD], n)
    kind[:, 1] = wl.WRITE_SLOT
    arg[:, 0] = rng.integers(-30, 6, n)
    arg[:, 1] = [wl.slot_arg(0, int(k), int(a)) for k, a in zip(rng.integers(-1, 3, n), rng.integers(-100, 100, n))]
    b = _batch(np.full(n, 2), row.ravel(), np.zeros(2 * n), kind.ravel(), arg.ravel())
    _check([wl.kv_table(rows, 1)], b, scheme, gaps=gaps)
