"""The engine's host side under failing copies and allocations, without a GPU.

libcc.so runs on a HIP runtime of host memory (tests/fake_hip), loaded before
it in a child process: allocations are counted against a capacity, a chosen
call fails, and kernels only write the results that the host reads.  What is
checked is the host's own work: which status a call returns, what stays
allocated, and that memory kept for later batches never makes a call fail.
"""
import os
import subprocess
import sys

import pytest

from helpers import ROOT

SETUP = r'''
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(FAKE, mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, ROOT)
from paper_2406_10158_amd import binding as B
fake.fake_capacity.argtypes = [ctypes.c_size_t]
fake.fake_used.restype = fake.fake_peak.restype = ctypes.c_size_t
fake.fake_fail.argtypes = [ctypes.c_char_p, ctypes.c_long]
fake.fake_batch.argtypes = [ctypes.c_uint64] * 3
MB = 1 << 20

def engine(rows=4096):
    fake.fake_reset()
    return B.Engine([np.zeros((rows, 1), np.int64)])

def submit(eng, scheme="occ", txns=256, ops=4, ordered=True):
    t = np.zeros(txns, B.TXN_DTYPE)
    t["first_op"], t["n_ops"] = np.arange(txns) * ops, ops
    return B.cc_submit_batch(eng.ctx, t, np.zeros(txns * ops, B.OP_DTYPE), B.SCHEMES[scheme])

def status(f, *a, **k):
    try:
        f(*a, **k)
    except B.CCError as e:
        return e.status
    return B.CC_OK
'''


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    from paper_2406_10158_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    lib = str(tmp_path_factory.mktemp("fake_hip") / "libfake.so")
    src = os.path.join(ROOT, "tests", "fake_hip", "fake_hip.cpp")
    r = subprocess.run([build.HIPCC, *build.COMMON, "-shared", src, "-o", lib], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(code):
        r = subprocess.run([sys.executable, "-c", f"ROOT, FAKE = {ROOT!r}, {lib!r}\n" + SETUP + code + "\nprint('ok')"],
                           capture_output=True, text=True, timeout=100, cwd=ROOT)
        assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
    return run


@pytest.mark.parametrize("scheme", ["occ", "tictoc", "gacco"])
def test_failed_copy_of_the_batch_is_reported(child, scheme):
    # of a context's first submission, small (from pinned memory) and large, and of a later one
    child(f'''
for txns in (256, 1 << 15):
    for copy in (0, 1):
        if txns == 256 and copy:
            continue  # one copy
        with engine() as eng:
            fake.fake_fail(b"hipMemcpyHtoD", copy)
            assert status(submit, eng, {scheme!r}, txns) == B.CC_E_HIP, (txns, copy)
            fake.fake_fail(b"", 0)
            B.cc_release_batch(eng.ctx, submit(eng, {scheme!r}, txns))
            fake.fake_fail(b"hipMemcpyHtoD", copy)
            assert status(submit, eng, {scheme!r}, txns) == B.CC_E_HIP, (txns, copy)
''')


@pytest.mark.parametrize("scheme", ["occ", "mvcc", "gputx"])
def test_a_failed_call_does_not_fail_the_next(child, scheme):
    # out of memory in a submission and in a run; the same calls then succeed
    child(f'''
for nth in range(8):
    with engine() as eng:
        fake.fake_fail(b"hipMalloc", nth)
        st = status(submit, eng, {scheme!r})
        fake.fake_fail(b"", 0)
        assert st in (B.CC_OK, B.CC_E_NOMEM), st
        bid = submit(eng, {scheme!r})
        fake.fake_fail(b"hipMalloc", 0)
        st = status(eng.run, bid)
        fake.fake_fail(b"", 0)
        assert st in (B.CC_OK, B.CC_E_NOMEM), st
        eng.run(bid)
''')


KEPT = r'''
def keep(eng):
    """Four released batches, whose arenas the context keeps, and the scratch of their submission."""
    for bid in [submit(eng, "gacco", 1 << 14, 16) for _ in range(4)]:
        B.cc_release_batch(eng.ctx, bid)

def room(megabytes):
    fake.fake_capacity(fake.fake_used() + int(megabytes * MB))
'''


@pytest.mark.parametrize("what,code", [
    ("submission scratch", """
    keep(eng)
    room(20)
    submit(eng, "occ", 1 << 16, 16)"""),
    ("arena", """
    keep(eng)
    room(1)
    submit(eng, "gacco", 1 << 16, 4)
    submit(eng, "mvcc", 256, 4)"""),
    ("breaks", """
    keep(eng)
    room(1)
    fake.fake_batch(0, 1, 0)
    submit(eng, "gacco", 1 << 14, 16)"""),
    ("hot-row engine's lists", """
    keep(eng)
    room(0.1)
    fake.fake_batch(1 << 24, 0, 1 << 16)
    assert eng.run(submit(eng, "occ", 1 << 14, 16))["engine_txns"] == 1 << 14"""),
    ("hot-row engine's scratch", """
    fake.fake_batch(1 << 24, 0, 1 << 20)
    bid = submit(eng, "occ", 1 << 14, 16)
    fake.fake_batch(0, 0, 0)
    keep(eng)
    room(10)
    assert eng.run(bid)["engine_txns"] == 1 << 14"""),
    ("version pointers", """
    bid = submit(eng, "mvcc")
    keep(eng)
    room(1)
    eng.run(bid)"""),
    ("rank states", """
    bid = submit(eng, "gputx")
    keep(eng)
    room(1)
    eng.run(bid)"""),
    ("latches", """
    bid = submit(eng, "tictoc")
    keep(eng)
    room(1)
    eng.run(bid, flags=B.CC_RUN_LATCH)"""),
    ("arrivals", """
    bid = submit(eng, "tictoc", 1 << 17, 1)
    keep(eng)
    room(1)
    B.cc_set_arrivals(eng.ctx, bid, np.arange(1 << 17))"""),
    ("index", """
    keep(eng)
    room(20)
    eng.create_index(0, np.arange(1 << 21))"""),
], ids=lambda v: v.replace(" ", "-") if "\n" not in v else "")
def test_kept_memory_makes_room(child, what, code):
    # with little room beside it, so that the call succeeds only with what the context keeps given back
    child(KEPT + "with engine(1 << 21) as eng:" + code + "\nassert fake.fake_used() == 0")


def test_released_batches_leave_at_most_what_the_header_says(child):
    # a hot-row engine of 40M operations, whose scratch is above the gibibyte that is kept
    child('''
with engine() as eng:
    used = fake.fake_used()
    fake.fake_batch(1 << 24, 0, 40 << 20)
    bid = submit(eng, "occ", 1 << 14, 16)
    for _ in range(2):
        peak = fake.fake_used()
        assert eng.run(bid)["engine_txns"] == 1 << 14
    assert peak - used > 1 << 30  # (kept for the batch's next run)
    B.cc_release_batch(eng.ctx, bid)
    assert fake.fake_used() - used <= 512 * MB
    for _ in range(6):  # five released batches of up to 250 MB
        fake.fake_batch(0, 0, 0)
        ids = [submit(eng, "gacco", 1 << 16, 32 + i) for i in range(5)]
        for b in ids:
            B.cc_release_batch(eng.ctx, b)
        assert fake.fake_used() - used <= (512 + 1024) * MB
assert fake.fake_used() == 0
''')


def test_tables_are_allocated_once_whatever_fails_behind_them(child):
    # the fills of the values and of the counts per row, failing one after the other
    child('''
fake.fake_reset()
for nth in range(3):
    ctx = B.cc_init()
    t = B.cc_create_table(ctx, 1 << 16, 4)
    rows = np.ones((1 << 16, 4), np.int64)
    fake.fake_fail(b"hipMemsetAsync", nth)
    st = status(B.cc_load, ctx, t, rows)
    fake.fake_fail(b"", 0)
    assert st in (B.CC_OK, B.CC_E_HIP), st
    B.cc_load(ctx, t, rows)
    B.cc_destroy(ctx)
    assert fake.fake_used() == 0, nth
''')
