"""A captured batch whose options changed since the call that sized the buffers.

Under capture nothing may be allocated, so the buffers have to be there: a
program solves once, then captures.  If it changes the grid in between (the
stack size or max_workgroups, with the queue's size unchanged) no buffer has
to grow, and the capture must be taken.  In a process of its own, because any
earlier solve of this one may have sized the buffers.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import sys
sys.path[:0] = [%r, %r]
import numpy as np
import torch
from test_gpu_graph import load_golden
from paper_1705_02843_amd import bpida as B

first, then = eval(sys.argv[1])
states, want_len, want_nodes = load_golden("c1_walk40")
states, want_len, want_nodes = states[:8], want_len[:8], want_nodes[:8]
d_states = torch.from_numpy(states).cuda()
d_len = torch.full((8,), -9, dtype=torch.int32, device="cuda")
d_nodes = torch.zeros((8, 64), dtype=torch.int64, device="cuda")
d_status = torch.zeros(8, dtype=torch.int32, device="cuda")
s = torch.cuda.Stream()

def solve(stream):
    return B.solve_device_async(d_states, d_len, d_nodes, d_status, stream=stream)

for k, v in first.items():
    B.set_option(k, v)
with torch.cuda.stream(s):
    assert solve(s) == B.OK
s.synchronize()
for k, v in then.items():
    B.set_option(k, v)
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, stream=s):
    rc = solve(torch.cuda.current_stream())
assert rc == B.OK, B.strerror(rc)
for rep in range(3):
    d_len.fill_(-9)
    d_nodes.fill_(7)
    d_status.fill_(0)
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert (d_status.cpu().numpy() == 1).all(), rep
    np.testing.assert_array_equal(d_len.cpu().numpy(), want_len)
    np.testing.assert_array_equal(d_nodes.cpu().numpy().view(np.uint64), want_nodes)
print("captured and replayed")
""" % (ROOT, os.path.join(ROOT, "tests"))


@pytest.mark.parametrize("first,then", [
    ({"max_workgroups": 64, "queue_capacity": 65536}, {"max_workgroups": 0}),
    ({}, {"lds_stack_capacity": 768}),
    ({"queue_capacity": 65536}, {"queue_capacity": 65536, "lds_stack_capacity": 512, "wg_size": 256}),
])
def test_capture_on_a_larger_grid(first, then):
    print("case: options %r, then captured with %r" % (first, then), flush=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, repr((first, then))], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "captured and replayed" in r.stdout
