"""Batches submitted with keys none of whose operations is on an indexed table.

Such a batch names its rows as any other does, so it runs as the same batch
submitted without keys: OCC's hot-row engine takes every transaction that
writes a row written more than once in THIS batch, whatever batch the context
saw before.
"""
import numpy as np
import pytest

from helpers import binding, check
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu


def _on_table_1(b):
    return wl.Batch(b.first_op, b.n_ops, b.row, np.ones_like(b.table), b.field, b.kind, b.arg)


def _engine_txns(b):
    w = b.kind != wl.READ
    hot = np.bincount(b.row[w].astype(np.int64), minlength=int(b.row.max()) + 1) > 1
    hit = np.zeros(b.n_txns, bool)
    hit[np.repeat(np.arange(b.n_txns), b.n_ops.astype(np.int64))[w & hot[b.row]]] = True
    return int(hit.sum())


# rows of table 1, transactions, their ops, skew: uniform has rows written more than once
# but none often enough for the engine's plan of the most written rows
SHAPES = {"uniform": (1 << 16, 1 << 17, 8, 0.0), "skewed": (1 << 16, 1 << 13, 16, 0.9)}


@pytest.mark.parametrize("before", ["nothing", "other rows", "other table"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_batch_by_row_submitted_with_keys(shape, before):
    b_ = binding()
    rows, n, ops, theta = SHAPES[shape]
    print(f"[gpu] keys without an indexed table: {shape}, before: {before}", flush=True)
    tables = [wl.kv_table(512, 1), wl.kv_table(rows, 1)]
    b = _on_table_1(wl.kv_batch(rows, 1, n, ops=ops, theta=theta, seed=21))
    with b_.Engine(tables) as eng:
        eng.create_index(0, np.arange(512) * 7 + 3)
        if before != "nothing":
            o = wl.kv_batch(512, 1, 2_000, ops=4, theta=0.9, seed=22)
            bid = eng.submit(_on_table_1(o) if before == "other rows" else o, "occ")
            b_.cc_release_batch(eng.ctx, bid)
        bid = eng.submit_keyed(b, np.zeros(b.total_ops, np.int64), "occ")
        st = eng.run(bid)
        out, reads = eng.outcomes(bid, b.n_txns, b.total_ops)
        final = eng.tables()
    rep = check(tables, b, out, reads, final)
    assert rep.ok, rep
    assert st["engine_txns"] == _engine_txns(b)


def test_engine_with_nothing_to_run():
    # no row written twice: no engine, by default or forced
    b_ = binding()
    tables = [wl.kv_table(512, 1), wl.kv_table(4_096, 1)]
    z = np.zeros(4_096)
    b = wl.Batch(np.arange(512, dtype=np.uint64) * np.uint64(8), np.full(512, 8, np.uint32),
                 np.random.default_rng(2).permutation(4_096).astype(np.uint32), np.ones(4_096, np.uint16),
                 z.astype(np.uint8), np.full(4_096, wl.ADD, np.uint8), np.ones(4_096, np.int64))
    with b_.Engine(tables) as eng:
        eng.create_index(0, np.arange(512))
        bid = eng.submit_keyed(b, np.zeros(b.total_ops, np.int64), "occ")
        for flags in (0, b_.CC_RUN_HOT_ENGINE):
            st = eng.run(bid, flags=flags)
            assert st["engine_txns"] == 0 and st["committed"] == 512
