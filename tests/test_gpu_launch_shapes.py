"""The library's choice of a launch shape, alone and beside the caller's wavefronts per workgroup.

A kernel's variant holds so many operations a lane that at most 4, 8 or 16
wavefronts fit.  With lanes_per_txn 0 the lanes follow the batch's contention,
and have to leave room for the caller's wavefronts whatever the contention and
however the batch came in: by row, by key, or through cc_run_static (in a child
process that initialises torch first: torch carries its own HIP runtime).
"""
import subprocess
import sys

import numpy as np
import pytest

from helpers import ROOT, SCHEMES, binding, check, run_and_check
from paper_2406_10158_amd import workload as wl

pytestmark = pytest.mark.gpu


def _flags(scheme):
    return binding().CC_RUN_NO_HOT_ENGINE if scheme == "occ" else 0


def _batch(share, ops):
    """20,000 transactions of up to `ops` operations on 200,000 rows, `share` of them also adding to row 0."""
    rng = np.random.default_rng(ops)
    b = wl.kv_batch(199_999, 1, 20_000, ops=(ops - 3, ops), theta=0.0, seed=ops)
    b.row[:] += 1
    at = b.first_op[rng.random(b.n_txns) < share].astype(np.int64)
    b.row[at], b.kind[at], b.arg[at] = 0, wl.ADD, 1
    return [wl.kv_table(200_000, 1)], b


@pytest.mark.parametrize("waves", [9, 16])
@pytest.mark.parametrize("share,ops", [(0.0, 4), (0.0, 16), (0.0, 33), (0.0, 64), (0.005, 16), (0.005, 33),
                                       (0.005, 64), (0.1, 33)])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_lanes_leave_room_for_the_callers_wavefronts(scheme, share, ops, waves):
    tabs, b = _batch(share, ops)
    run_and_check(tabs, b, scheme, waves_per_wg=waves, flags=_flags(scheme))


@pytest.mark.parametrize("rows,ops", [(300, 4), (300, 5), (4_096, 16), (4_096, 17), (20_000, 64), (20_000, 65),
                                      (262_144, 64), (2_000_000, 64)])
@pytest.mark.parametrize("read_ratio", [0.1, 0.5, 0.9])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_shapes_by_the_counted_conflicts(scheme, read_ratio, rows, ops):
    # on both sides of the numbers of operations and of the conflicts at which the shape changes
    tabs, b = wl.kv_workload(n_rows=rows, n_fields=1, n_txns=3_000, ops=(max(1, ops - 30), ops), theta=0.0,
                             read_ratio=read_ratio, seed=rows + ops)
    run_and_check(tabs, b, scheme)
    if scheme == "occ":
        run_and_check(tabs, b, scheme, flags=_flags(scheme))


@pytest.mark.parametrize("waves", [9, 16])
@pytest.mark.parametrize("n", [4_096, 4_097, 20_000])
def test_keyed_batch(n, waves):
    b_ = binding()
    tabs = [wl.kv_table(1_000_000, 1)]
    b = wl.kv_batch(1_000_000, 1, n, ops=16, theta=0.0, seed=n)
    keys = np.arange(1_000_000) * 3 + 1
    with b_.Engine(tabs) as eng:
        eng.create_index(0, keys)
        bid = eng.submit_keyed(b, wl.keyed_ops(b, [keys]), "tictoc")
        for _ in range(2):  # the second with the rows counted behind the first
            eng.load(tabs)
            eng.run(bid, waves_per_wg=waves)
            out, reads = eng.outcomes(bid, b.n_txns, b.total_ops)
            rep = check(tabs, b, out, reads, eng.tables())
            assert rep.ok, rep


CHILD = r'''
import sys
import torch
torch.cuda.init()
sys.path.insert(0, ROOT)
import numpy as np
from paper_2406_10158_amd import binding as B, workload as wl
import oracle

def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8)).to("cuda")

tabs = [wl.kv_table(200_000, 1)]
with B.Engine(tabs) as eng:
    for ops in (4, 16, 33):
        b = wl.kv_batch(200_000, 1, 10_000, ops=ops, theta=0.0, seed=ops)
        for waves in (9, 16):
            print(f"[child] {ops} ops, {waves} wavefronts", flush=True)
            eng.load(tabs)
            txns, rec = B.pack_batch(b)
            out = torch.zeros(b.n_txns * B.OUTCOME_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
            reads = torch.zeros(b.total_ops, dtype=torch.int64, device="cuda")
            B.cc_run_static(eng.ctx, dev(txns), dev(rec), B.CC_OCC, B.run_params(waves_per_wg=waves), out, reads)
            torch.cuda.synchronize()
            o = out.cpu().numpy().view(B.OUTCOME_DTYPE)
            rep = oracle.check_run(tabs, b, o["status"], o["serial_hi"], o["serial_lo"], reads.cpu().numpy(), eng.tables())
            assert rep.ok, rep
print("child ok", flush=True)
'''


def test_static_run():
    r = subprocess.run([sys.executable, "-c", f"ROOT = {ROOT!r}\n" + CHILD], capture_output=True, text=True,
                       timeout=110, cwd=ROOT)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr
