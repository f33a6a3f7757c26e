"""The chain scan on one cell's long chain with constant slot writes in it.

A slot write that multiplies its source by 0 gives the tile it lies in a total
that does not depend on the tiles before, so that the tile the chain ends in
may store the cell while the one it begins in still has its load to make; the
scan orders the two (tests/test_chain_model.py is the model of how).  Here
chains of more than three tiles of 2,048 accesses, with constants in the middle
tiles, in all of them, and after conditional adds, which are breaks; read
values and cells are compared with a replay in serial order.
"""
import numpy as np
import pytest

import oracle
from helpers import binding, check
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu
TILE = 2048


def _batch(kind, arg, rng):
    """Per access of the hot cell (row 1) one transaction; constants take their source from a row of their own."""
    n = len(kind)
    const = kind == wl.WRITE_SLOT
    n_ops = np.where(const, 2, 1).astype(np.uint32)
    first = (np.cumsum(n_ops) - n_ops).astype(np.uint64)
    m = int(n_ops.sum())
    row, k, a = np.ones(m, np.uint32), np.zeros(m, np.uint8), np.zeros(m, np.int64)
    hot = first.astype(np.int64) + const
    k[hot] = kind
    a[hot] = arg
    row[first[const].astype(np.int64)] = 2 + rng.integers(0, 50, int(const.sum()))
    z = np.zeros(m)
    return wl.Batch(first, n_ops, row, z.astype(np.uint16), z.astype(np.uint8), k, a)


@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("scheme", ["gacco", "gputx", "occ"])
@pytest.mark.parametrize("kinds", ["middle", "every tile", "after breaks", "one"])
def test_constants_inside_a_long_chain(kinds, scheme, strict):
    if scheme == "gputx" and strict:
        pytest.skip("the scan is the one of gacco; the rank pass has no constants")
    b_ = binding()
    rng = np.random.default_rng(5)
    n = 9 * TILE + 77
    kind, arg = np.where(rng.random(n) < 0.3, wl.READ, wl.ADD), rng.integers(-30, 31, n)
    at = {"middle": rng.integers(3 * TILE, 6 * TILE, 40), "every tile": rng.integers(0, n, 300),
          "after breaks": rng.integers(4 * TILE, 6 * TILE, 20), "one": np.array([4 * TILE + 1])}[kinds]
    if kinds == "after breaks":
        kind[rng.integers(TILE, 3 * TILE, 200)] = wl.COND_ADD
    kind[at] = wl.WRITE_SLOT
    arg[at] = [wl.slot_arg(0, 0, int(v)) for v in rng.integers(-1000, 1000, len(at))]
    arg[kind == wl.READ] = 0
    b = _batch(kind, arg, rng)
    tables = [wl.kv_table(60, 1)]
    print(f"[gpu] chain constants {kinds} {scheme} strict={strict} ops={b.total_ops}", flush=True)
    flags = (b_.CC_RUN_STRICT_FENCES if strict else 0) | (b_.CC_RUN_HOT_ENGINE if scheme == "occ" else 0)
    with b_.Engine(tables) as eng:
        bid = eng.submit(b, scheme)
        st = eng.run(bid, flags=flags)
        out, reads = eng.outcomes(bid, b.n_txns, b.total_ops)
        final = eng.tables()
    if scheme == "occ":
        # every write of the hot row's in the engine; reads of it may come after
        assert st["engine_txns"] >= int((kind != wl.READ).sum())
        rep = check(tables, b, out, reads, final)
        assert rep.ok, rep
        return
    exp_fin, exp_reads = oracle.id_order_expected(tables, b)
    assert np.all(out["status"] == oracle.COMMITTED)
    assert np.array_equal(reads, exp_reads)
    assert all(np.array_equal(g, e) for g, e in zip(final, exp_fin))
