"""What bench.py counts to OCC's hot-row engine: its transactions, and their accesses by hand."""
import numpy as np

from paper_2406_10158_amd import workload as wl
from test_bench_accounting import _batch, bench


def test_engine_transactions_are_the_first_tickets():
    # tickets start at 1: a batch of six, of which the engine ran four in the order 2, 0, 5, 3
    tickets = np.array([2, 5, 1, 4, 6, 3], np.uint64)
    assert bench.engine_transactions(tickets, 4).tolist() == [0, 2, 3, 5]
    assert bench.engine_transactions(tickets, 6).tolist() == list(range(6))
    assert len(bench.engine_transactions(tickets, 0)) == 0


def test_engine_counts_of_a_small_batch():
    # row 7 field 0 written twice and read once, row 7 field 1 read, row 9 written: 5 ops, 3 cells, 2 written
    b = _batch([[(0, 7, 0, wl.ADD, 1), (0, 9, 0, wl.ADD, 2)], [(0, 7, 0, wl.ADD, 5), (0, 7, 1, wl.READ, 0)],
                [(0, 7, 0, wl.READ, 0)]])
    cnt = bench.engine_counts(b, 1 << 16)
    assert cnt["passes"] == 2 and bench.engine_counts(b, (1 << 16) + 1)["passes"] == 3
    assert cnt["random_loads"] == 5 + 3 and cnt["random_stores"] == 5 + 2
    assert cnt["stream_bytes"] == 5 * (40 + 2 * 20 + 8) + 3 * 48
    assert cnt["bytes"] == 5 * 24 + 3 * 8 + 2 * 8 + 3 * 40
    # the seconds are the counts at the probed rates
    probes = {"gather_880MB_Gops": 50.0, "scatter_880MB_Gops": 25.0, "stream_GBps": 4000.0}
    t = 8 / 50e9 + 7 / 25e9 + cnt["stream_bytes"] / 4e12
    assert abs(bench.engine_seconds(cnt, probes) - t) < 1e-15
