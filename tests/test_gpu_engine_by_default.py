"""cc_engine_plan's by_default against what cc_run does with the batch.

Batches that meet much or little, with the writes of the most written rows far
above the rest's or level with them: the answer is whether a run without flags
uses the hot-row engine.
"""
import numpy as np
import pytest

from helpers import binding
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu

# rows, transactions, ops, skew, and whether the engine runs by default
BATCHES = {
    "headline-like": (200_000, 1 << 15, 16, 0.9, True),
    "uniform, contended": (1 << 16, 1 << 17, 16, 0.0, True),      # no row stands out
    "uniform, uncontended": (1 << 20, 1 << 12, 4, 0.0, False),
    "a few transactions": (4, 60, 1, 0.0, False),                 # every row in the plan, nothing to gain
    "no row twice": (1 << 20, 64, 4, 0.0, False),
}


@pytest.mark.parametrize("case", list(BATCHES))
def test_by_default_says_what_a_run_does(case):
    b_ = binding()
    rows, n, ops, theta, exp = BATCHES[case]
    tables = [wl.kv_table(rows, 1)]
    b = wl.kv_batch(rows, 1, n, ops=ops, theta=theta, seed=31)
    print(f"[gpu] engine by default: {case}", flush=True)
    with b_.Engine(tables) as eng:
        bid = eng.submit(b, "occ")
        plan, n_plan, by_default = b_.cc_engine_plan(eng.ctx, bid)
        st = eng.run(bid)
        assert by_default == (st["engine_txns"] > 0) == exp
        w = b.kind != wl.READ
        owner = np.repeat(np.arange(b.n_txns), b.n_ops.astype(np.int64))
        assert n_plan == len(np.unique(owner[w & np.isin(b.row, plan)]))
        again = b_.cc_engine_plan(eng.ctx, bid)
        assert np.array_equal(again[0], plan) and again[1:] == (n_plan, by_default)
        assert eng.run(bid, flags=b_.CC_RUN_NO_HOT_ENGINE)["engine_txns"] == 0
