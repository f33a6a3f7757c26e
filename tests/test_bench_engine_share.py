"""Which transactions bench.py counts to OCC's hot-row engine."""
import numpy as np

from test_bench_accounting import bench


def test_engine_transactions_are_the_first_tickets():
    # tickets start at 1: a batch of six, of which the engine ran four in the order 2, 0, 5, 3
    tickets = np.array([2, 5, 1, 4, 6, 3], np.uint64)
    assert bench.engine_transactions(tickets, 4).tolist() == [0, 2, 3, 5]
    assert bench.engine_transactions(tickets, 6).tolist() == list(range(6))
    assert len(bench.engine_transactions(tickets, 0)) == 0
