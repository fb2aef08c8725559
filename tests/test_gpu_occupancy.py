"""The search kernels keep the occupancy their stacks allow.

Waves a compute unit, as the persistent grid shows them: 16-node rounds up to
5 a SIMD, 64-node rounds what the stack's LDS allows, up to 6.  And the 16-node
rounds' results, first solutions too, against the stored oracle results.
"""
import numpy as np
import pytest

from test_gpu_first_solution import check_first_solution
from test_gpu_parity import B, assert_parity, load_golden, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npl,cap,waves", [(16, 128, 20), (16, 256, 20), (16, 512, 20), (16, 1024, 16), (16, 2048, 8),
                                           (64, 512, 24), (64, 640, 24), (64, 672, 24), (64, 768, 20), (64, 1024, 16)])
def test_waves_per_compute_unit(opts, npl, cap, waves):
    import torch
    B = opts
    set_mode(B, "batched")
    print("case: %d-node rounds, %d entries" % (npl, cap), flush=True)
    states, length, nodes = load_golden("c1_walk40")
    B.set_option("nodes_per_round", npl)
    B.set_option("lds_stack_capacity", cap)
    rc, ln, got = B.solve_raw(states, 4)
    assert rc == B.OK
    assert_parity(ln, got, length, nodes)
    assert B.last_stats()["grid"] >= waves * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("cap,wg", [(256, 64), (512, 64), (512, 128), (512, 256)])
def test_small_stacks_keep_their_registers(opts, cap, wg):
    """256 and 512 entries leave LDS for 8 waves a SIMD, whose registers would be spilled: 6."""
    import torch
    B = opts
    set_mode(B, "batched")
    print("case: 64-node rounds, %d entries, workgroups of %d" % (cap, wg), flush=True)
    B.set_option("lds_stack_capacity", cap)
    B.set_option("wg_size", wg)
    goal = np.arange(9, dtype=np.uint8)[None]
    rc, ln, _ = B.solve_raw(goal, 3)
    assert rc == B.OK and ln[0] == 0
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert B.last_stats()["grid"] * (wg // 64) == 24 * cus


@pytest.mark.parametrize("cap", [128, 512, 1024])
def test_16_node_rounds_back_to_back(opts, cap):
    B = opts
    set_mode(B, "batched16")
    B.set_option("lds_stack_capacity", cap)
    states, length, nodes = load_golden("c2_md30_38")
    states, length, nodes = states[:12], length[:12], nodes[:12]
    print("case: 12 hard states, %d entries" % cap, flush=True)
    rc, ln, got = B.solve_raw(states, 4)
    assert rc == B.OK
    assert_parity(ln, got, length, nodes)
    B.set_option("first_solution", 1)
    rc, ln, got = B.solve_raw(states, 4)
    assert rc == B.OK
    check_first_solution(ln, got, length, nodes, "16-node rounds")
