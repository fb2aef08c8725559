"""A limit's roots, and a busy wave's oldest entries, dealt to several waves.

Hard states one at a time, with a whole grid waiting, so that every limit of
4096, 8192 and 16384 nodes and more is dealt 2, 4 and 8 ways; split depths
whose root lists leave chunks of every remainder, chunks of 16 to 64 roots (a
chunk of no more roots than waves is not dealt), and the smallest ring, whose
slots the parts of one push wrap around.  Exact against the oracle.
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


@pytest.mark.parametrize("depth,chunk,queue", [(0, 64, 0), (1, 64, 64), (2, 64, 0), (3, 16, 0), (4, 32, 64), (5, 64, 64),
                                               (6, 64, 0), (8, 16, 64), (8, 64, 0)])
def test_dealt_limits_are_exact(opts, depth, chunk, queue):
    B = opts
    set_mode(B, "batched")
    B.set_option("frontier_depth", depth)
    B.set_option("queue_chunk", chunk)
    B.set_option("queue_capacity", queue)
    for name, width in (("c2_md30_38", 4), ("c4_mixed_w5", 5)):
        states, length, nodes = load(name)
        for k in range(3):
            print("case: %s[%d], depth %d, chunk %d, queue %d" % (name, k, depth, chunk, queue), flush=True)
            rc, ln, got = B.solve_raw(states[k:k + 1], width)
            assert rc == B.OK, B.strerror(rc)
            assert_parity(ln, got, length[k:k + 1], nodes[k:k + 1], name)
