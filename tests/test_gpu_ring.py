"""The batched 64-node rounds: stacks of entries with moves left.

One f-limit far above the heuristic, so that slack runs deep and a root may
keep all four moves: the count of that limit against a layer-by-layer path
count (tests/puzzle_ref.py), exactly.  Split depths 0 (one root, all its
moves), 1 and 5, the smallest and largest stacks of each width, and one
workgroup that spills as well as a full grid.
"""
import functools

import numpy as np
import pytest

import puzzle_ref as R
from test_gpu_parity import B, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu

# width, stack, split depth, moves from the goal, limit above the first one
CASES = [(3, 256, 0, 4, 28), (3, 256, 5, 9, 24), (3, 512, 1, 12, 22), (3, 2048, 0, 1, 28),
         (4, 512, 0, 10, 16), (4, 512, 5, 6, 18), (4, 640, 1, 14, 14), (4, 672, 0, 3, 20),
         (4, 768, 1, 9, 16), (4, 2048, 0, 10, 16),
         (5, 1024, 0, 12, 12), (5, 1024, 6, 24, 10), (5, 2048, 1, 30, 10)]


@functools.lru_cache(maxsize=None)
def count_at(start, width, limit):
    return R.layered_path_count(start, width, limit)


@pytest.mark.parametrize("maxwg", [1, 0])
@pytest.mark.parametrize("width,cap,depth,walk,above", CASES)
def test_count_of_one_high_limit(opts, width, cap, depth, walk, above, maxwg):
    from paper_1705_02843_amd import instances as I
    B = opts
    set_mode(B, "batched")
    rng = np.random.Generator(np.random.PCG64(1000 * width + walk))
    states = np.stack([I.random_walk(rng, width, walk)[0] for _ in range(3)])
    print("case: %dx%d, stack %d, depth %d, walk %d, limit +%d" % (width, width, cap, depth, walk, above), flush=True)
    B.set_option("lds_stack_capacity", cap)
    B.set_option("frontier_depth", depth)
    B.set_option("max_workgroups", maxwg)
    for s in states:
        start = tuple(int(x) for x in s)
        limit = R.manhattan(start, width) + above
        B.set_option("start_threshold", limit)
        rc, ln, nodes = B.solve_raw(s[None], width)
        assert rc == B.OK, B.strerror(rc)
        assert ln[0] == limit  # the walk is shorter: the limit holds a goal
        want = count_at(start, width, limit)
        assert int(nodes[0, above // 2]) == want
        assert int(nodes[0].sum()) == want
