"""End of a search with many more waves than work.

Thousands of waves wait on queue tickets, far more than the ring has slots
when it is small, and leave when the last instance completes; batches of one
state, of invalid states only, and of fewer and more states than waves.
Exact against the stored oracle results, and ended by the last instance, not
by the idle watchdog (whose period here is longer than the test allows).
"""
import time

import numpy as np
import pytest

from test_gpu_parity import B, assert_parity, load_golden, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,queue,maxwg", [(1, 64, 0), (1, 0, 0), (8, 64, 0), (64, 0, 0), (64, 0, 31), (64, 1024, 33)])
def test_waiting_waves_leave_with_the_last_instance(opts, n, queue, maxwg):
    B = opts
    set_mode(B, "batched")
    print("case: %d states, queue %d, grid %d" % (n, queue, maxwg), flush=True)
    states, length, nodes = load_golden("c1_walk40")
    B.set_option("queue_capacity", queue)
    B.set_option("max_workgroups", maxwg)
    B.set_option("watchdog_ms", 20000)
    for _ in range(3):
        t = time.time()
        rc, ln, got = B.solve_raw(states[:n])
        assert rc == B.OK, B.strerror(rc)
        assert time.time() - t < 10.0
        assert_parity(ln, got, length[:n], nodes[:n], "n=%d" % n)


def test_batch_with_nothing_to_search(opts):
    B = opts
    set_mode(B, "batched")
    bad = np.zeros((5, 16), np.uint8)
    t = time.time()
    rc, ln, got = B.solve_raw(bad)
    assert rc == B.EINVAL and (ln == -1).all() and not got.any()
    assert time.time() - t < 10.0
