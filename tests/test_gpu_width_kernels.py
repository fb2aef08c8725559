"""Batches of one width run a kernel without the other widths' rounds.

The same states as a batch of one width and through the mixed-width call (the
kernel that holds every round) give the same lengths and counts, both the
stored oracle's: every stack size that has such kernels, all solutions and
first solution, a full grid and a few waves.
"""
import json
import os

import numpy as np
import pytest

from test_gpu_parity import B, assert_parity, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


def load(name):
    with open(os.path.join(os.path.dirname(__file__), "golden", name + ".json")) as f:
        recs = json.load(f)["instances"]
    # (one hex digit a cell up to 4x4, two for 5x5)
    states = np.array([[int(c, 16) for c in r["state"]] if len(r["state"]) <= 16 else list(bytes.fromhex(r["state"]))
                       for r in recs], np.uint8)
    nodes = np.zeros((len(recs), 64), np.uint64)
    for i, r in enumerate(recs):
        nodes[i, :len(r["nodes"])] = r["nodes"]
    return states, np.array([r["length"] for r in recs], np.int32), nodes


GOLDEN = {3: ("c4_mixed_w3", 200), 4: ("c1_walk40", 40), 5: ("c4_mixed_w5", 6)}


def states_of(width):
    name, n = GOLDEN[width]
    states, length, nodes = load(name)
    order = np.argsort(nodes.astype(np.float64).sum(axis=1))[:n]
    return np.ascontiguousarray(states[order]), length[order], nodes[order]


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("maxwg", [0, 3])
@pytest.mark.parametrize("width,cap", [(w, c) for w in (3, 4, 5) for c in (256, 512, 640, 672, 768, 1024, 2048)
                                       if c >= (256, 512, 1024)[w - 3]])
def test_one_width_and_mixed_agree(opts, width, cap, maxwg, first):
    B = opts
    set_mode(B, "batched")
    B.set_option("lds_stack_capacity", cap)
    B.set_option("max_workgroups", maxwg)
    print("case: %dx%d, stack %d, grid %d, first %d" % (width, width, cap, maxwg, first), flush=True)
    states, length, nodes = states_of(width)
    B.set_option("first_solution", first)
    try:
        rc, ln, got = B.solve_raw(states, width)
        assert rc == B.OK, B.strerror(rc)
        rc2, ln2, got2 = B.solve_mixed_raw([s.reshape(-1) for s in states])
        assert rc2 == B.OK, B.strerror(rc2)
    finally:
        B.set_option("first_solution", 0)
    for l, g in ((ln, got), (ln2, got2)):
        if not first:
            assert_parity(l, g, length, nodes, "%dx%d" % (width, width))
            continue
        assert (l == length).all()
        for i in range(len(l)):  # the limits before the last are searched whole
            last = int(np.flatnonzero(nodes[i])[-1]) if nodes[i].any() else 0
            assert (g[i, :last] == nodes[i, :last]).all() and not g[i, last + 1:].any()
            assert g[i, last] <= nodes[i, last]
