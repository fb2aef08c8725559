"""Dealing a limit's roots leaves the queue room for the rest.

A queue that holds the chunks of 64 roots and what the stacks spill must stay
enough when limits are dealt out.  A deep split on a small grid has thousands
of root chunks and few waves to take them; a push that finds its slot taken
gives up at once here (push_spin 1), so a queue that fills up for a moment
shows as BPIDA_ENOMEM.  And with a queue of 64 slots under a full grid, where
any push may find its slot taken: exact, or BPIDA_ENOMEM, but never short
counts, and the next call is exact again.
"""
import pytest

from test_gpu_deal import load
from test_gpu_parity import B, assert_parity, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,width,depth,k", [("c2_md30_38", 4, 14, 0), ("c2_md30_38", 4, 16, 1),
                                                ("c4_mixed_w5", 5, 12, 0), ("c4_mixed_w5", 5, 12, 2)])
def test_deep_split_on_a_small_grid(opts, name, width, depth, k):
    B = opts
    set_mode(B, "batched")
    states, length, nodes = load(name)
    print("case: %s[%d], depth %d, 16 workgroups" % (name, k, depth), flush=True)
    B.set_option("frontier_depth", depth)
    B.set_option("max_workgroups", 16)
    B.set_option("push_spin", 1)
    rc, ln, got = B.solve_raw(states[k:k + 1], width)
    assert rc == B.OK, B.strerror(rc)
    assert_parity(ln, got, length[k:k + 1], nodes[k:k + 1], name)


@pytest.mark.parametrize("depth", [2, 8])
def test_refused_chunks_never_shorten_counts(opts, depth):
    B = opts
    set_mode(B, "batched")
    states, length, nodes = load("c2_md30_38")
    B.set_option("frontier_depth", depth)
    for k in range(3):
        print("case: c2_md30_38[%d], depth %d, 64 slots, no waiting for a slot" % (k, depth), flush=True)
        B.set_option("queue_capacity", 64)
        B.set_option("push_spin", 1)
        rc, ln, got = B.solve_raw(states[k:k + 1], 4)
        assert rc in (B.OK, B.ENOMEM)
        if rc == B.OK:
            assert_parity(ln, got, length[k:k + 1], nodes[k:k + 1], "64 slots")
        B.set_option("queue_capacity", 0)
        B.set_option("push_spin", 65536)
        rc, ln, got = B.solve_raw(states[k:k + 1], 4)
        assert rc == B.OK
        assert_parity(ln, got, length[k:k + 1], nodes[k:k + 1], "after it")


@pytest.mark.parametrize("queue", [64, 128, 256, 4096])
def test_small_queues_on_a_small_grid(opts, queue):
    """16 workgroups: from 128 slots (8 a wave) on a limit is dealt out while the queue is a quarter full."""
    B = opts
    set_mode(B, "batched")
    states, length, nodes = load("c2_md30_38")
    print("case: c2_md30_38[0..5], 16 workgroups, %d slots" % queue, flush=True)
    B.set_option("max_workgroups", 16)
    B.set_option("queue_capacity", queue)
    rc, ln, got = B.solve_raw(states[:6], 4)
    assert rc == B.OK, B.strerror(rc)
    assert_parity(ln, got, length[:6], nodes[:6], "%d slots" % queue)


@pytest.mark.parametrize("name,width,depth", [("c2_md30_38", 4, 10), ("c2_md30_38", 4, 14), ("c4_mixed_w5", 5, 8),
                                              ("c4_mixed_w5", 5, 12)])
def test_a_deep_split_is_not_dealt(opts, name, width, depth):
    """More than 768 roots make chunks enough: no more are taken than 64 roots each and what stacks push."""
    B = opts
    set_mode(B, "batched")
    states, length, nodes = load(name)
    print("case: %s[0], depth %d" % (name, depth), flush=True)
    B.set_option("frontier_depth", depth)
    rc, ln, got = B.solve_raw(states[:1], width)
    assert rc == B.OK
    assert_parity(ln, got, length[:1], nodes[:1], name)
    s = B.last_stats()
    limits = int((nodes[0] > 0).sum())
    assert s["chunks_popped"] <= s["roots_read"] // 64 + limits + s["chunks_pushed"]
