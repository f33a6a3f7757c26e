"""The transaction kernel's rounds and queue where they can go wrong.

Timestamp ordering, its multi-version form and TicToc on small tables whose
row groups mix read and written fields (operations that follow an earlier one
on their row), mostly reading, so that rows change between an attempt's look at
their words and its claim of them; batches whose size is around what a few
teams claim from the queue at a time; OCC's hot-row engine chosen by the
counted conflicts, with and without operations a scan cannot see through.
"""
import numpy as np
import pytest

import oracle
from helpers import binding, check, run_and_check
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("read", [0.5, 0.9])
@pytest.mark.parametrize("lanes", [1, 4, 16, 64])
@pytest.mark.parametrize("scheme", ["to", "mvcc", "tictoc"])
def test_row_groups_under_contention(scheme, lanes, read):
    print(f"[gpu] rounds {scheme} L={lanes} read={read}", flush=True)
    p = (1 - read) / 3
    tabs, b = wl.mixed_workload(n_txns=1_500, kind_p=(read, p, p, p), seed=17)
    run_and_check(tabs, b, scheme, lanes_per_txn=lanes)


@pytest.mark.parametrize("scheme", ["occ", "mvcc", "2pl_wd"])
@pytest.mark.parametrize("n", [1, 127, 128, 129, 383, 511, 512, 517])
def test_batches_around_a_claim(n, scheme):
    # four teams of 16 lanes: from 128 transactions on each comes back 32 times, and from 256 on
    # claims two at a time, from 512 on four
    b_ = binding()
    flags = b_.CC_RUN_NO_HOT_ENGINE if scheme == "occ" else 0
    print(f"[gpu] claims {scheme} n={n}", flush=True)
    tabs, b = wl.kv_workload(n_rows=300, n_fields=2, n_txns=n, ops=(1, 16), theta=0.5, seed=n)
    run_and_check(tabs, b, scheme, lanes_per_txn=16, waves_per_wg=1, grid=1, flags=flags)


@pytest.mark.parametrize("kind_p", [(0.5, 0.5, 0, 0), (0.4, 0.3, 0.3, 0), (0.35, 0.3, 0.2, 0.15)])
@pytest.mark.parametrize("n", [600, 1023, 1024, 1025, 2049])
def test_hot_engine_by_counted_conflicts(n, kind_p):
    print(f"[gpu] engine n={n} kinds={kind_p}", flush=True)
    tabs, b = wl.mixed_workload(n_txns=n, kind_p=kind_p, seed=n)
    st = run_and_check(tabs, b, "occ")[3]
    assert st["engine_txns"] > 0


@pytest.mark.parametrize("theta", [0.0, 0.9])
@pytest.mark.parametrize("n", [4096, 4097, 9000])
def test_keyed_batch_counted_at_its_first_run(n, theta):
    # more than 4,096 transactions: the rows the lookup found are counted behind it; the launch shape
    # then goes by them, and the counts are 0 again for the submission that follows
    b_ = binding()
    print(f"[gpu] keyed count n={n} theta={theta}", flush=True)
    tabs, b = wl.kv_workload(n_rows=5_000, n_fields=2, n_txns=n, ops=4, theta=theta, seed=n)
    keys = wl.index_keys(5_000, seed=3)
    op_keys = wl.keyed_ops(b, [keys])
    rb = oracle.with_rows(b, oracle.resolve_keys([keys], b, op_keys))
    with b_.Engine(tabs) as eng:
        eng.create_index(0, keys)
        bid = eng.submit_keyed(b, op_keys, "to")
        for _ in range(2):
            eng.load(tabs)
            eng.run(bid)
            out, reads = eng.outcomes(bid, b.n_txns, b.total_ops)
            rep = check(tabs, rb, out, reads, eng.tables())
            assert rep.ok, rep
        st = eng.run(eng.submit(b, "to"))
    assert st["hot_writes"] == wl.hottest_row_writes(b)[1]


@pytest.mark.parametrize("n", [3, 255, 511, 512, 513])
def test_percentiles_around_the_direct_ranks(n):
    # up to 512 transactions every latency counts those below it; 513 go through the histograms
    print(f"[gpu] direct ranks n={n}", flush=True)
    tabs, b = wl.kv_workload(n_rows=2_000, n_fields=2, n_txns=n, ops=4, theta=0.5, seed=n)
    with binding().Engine(tabs) as eng:
        bid = eng.submit(b, "2pl_nw")
        st = eng.run(bid)
        out, _ = eng.outcomes(bid, n, 0)
    lat = np.sort(out["commit_ns"])
    assert [st["lat_p50_ns"], st["lat_p99_ns"]] == [int(lat[int(q * (n - 1) + 0.5)]) for q in (0.5, 0.99)]
