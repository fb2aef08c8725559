"""A host-buffer call that is refused returns no answers of an earlier call.

Every host entry keeps its device buffers for the next call.  A call refused
before its launches (a stack its width cannot run on, plain mode on another
width than 4) must return lengths -1, counts 0 and no moves, whatever a solved
call before it left in those buffers; below and above the largest batch whose
results come through pinned memory (4096 states).
"""
import numpy as np
import pytest

from test_gpu_parity import B, load_golden, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


def nothing(length, nodes):
    assert (length == -1).all()
    assert (nodes == 0).all()


@pytest.mark.parametrize("n", [1, 64, 4097])
@pytest.mark.parametrize("entry", ["plain, 3x3", "batched, small stack", "mixed, small stack"])
def test_refused_solve_returns_nothing(opts, entry, n):
    B = opts
    set_mode(B, "batched")
    print("case: %s, %d states" % (entry, n), flush=True)
    states, want, _ = load_golden("c1_walk40")
    states = np.resize(states, (n, 16))
    rc, length, nodes = B.solve_raw(states, 4)
    assert rc == B.OK and (length == np.resize(want, n)).all() and nodes.any()
    if entry == "plain, 3x3":
        set_mode(B, "plain")
        goal = np.tile(np.arange(9, dtype=np.uint8), (n, 1))
        rc, length, nodes = B.solve_raw(goal, 3)
    else:
        B.set_option("lds_stack_capacity", 256)
        if entry == "batched, small stack":
            rc, length, nodes = B.solve_raw(states, 4)
        else:
            rc, length, nodes = B.solve_mixed_raw(list(states))
    assert rc == B.EINVAL
    nothing(length, nodes)


def test_refused_paths_return_nothing(opts):
    B = opts
    set_mode(B, "batched")
    print("case: paths on a small stack", flush=True)
    states, want, _ = load_golden("c1_walk40")
    rc, length, _, path = B.solve_paths_raw(states, 4)
    assert rc == B.OK and (length == want).all() and (path[:, 0] != 0xFF).all()
    B.set_option("lds_stack_capacity", 256)
    rc, length, nodes, path = B.solve_paths_raw(states, 4)
    assert rc == B.EINVAL
    nothing(length, nodes)
    assert (path == 0xFF).all()
