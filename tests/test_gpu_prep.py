"""The launch before a batched search: validation of every state on the device.

Random permutations, unsolvable ones and broken ones (a tile out of range, a
duplicate, no blank) of each width, with a limit cap below any heuristic so
that nothing is searched: every status as the parity rule says, lengths -1
and no counts; odd batch sizes, and the widths mixed in one launch.
"""
import numpy as np
import pytest

import puzzle_ref as R
from test_gpu_parity import B, opts, set_mode  # noqa: F401

pytestmark = pytest.mark.gpu


def states_and_status(width, n, rng):
    cells = width * width
    out, want = [], []
    for k in range(n):
        s = rng.permutation(cells).astype(np.uint8)
        blank = int(np.nonzero(s == 0)[0][0])
        ok = R.inversion_parity(tuple(int(x) for x in s)) == (blank // width + blank % width) % 2
        st = -3 if ok else -2
        if k % 4 == 3:
            p, how = rng.integers(cells), k // 4 % 4
            s[p] = (cells, 255, s[(p + 1) % cells], 31)[how]
            if how == 2 or int(s[p]) >= cells:
                st = -1
        out.append(s)
        want.append(st)
    return np.stack(out), np.array(want, np.int32)


@pytest.mark.parametrize("width,n", [(3, 1), (3, 129), (4, 1), (4, 63), (4, 300), (5, 1), (5, 77)])
def test_status_of_every_state(opts, width, n):
    import torch
    B = opts
    set_mode(B, "batched")
    B.set_option("max_threshold", 0)
    states, want = states_and_status(width, n, np.random.default_rng(100 * width + n))
    d = torch.from_numpy(states).cuda()
    ln = torch.full((n,), 5, dtype=torch.int32, device="cuda")
    nd = torch.full((n, 64), 5, dtype=torch.int64, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    for call in (B.solve_device_async, B.solve_device_noalloc):
        assert call(d, ln, nd, st, width=width) == B.OK
        torch.cuda.synchronize()
        assert (st.cpu().numpy() == want).all()
        assert (ln == -1).all() and (nd == 0).all()


def test_status_mixed_widths(opts):
    B = opts
    set_mode(B, "batched")
    B.set_option("max_threshold", 0)
    rng = np.random.default_rng(9)
    parts = [states_and_status(w, 9, rng) for w in (5, 3, 4)]
    states = [s for p, _ in parts for s in p]
    want = np.concatenate([w for _, w in parts])
    order = rng.permutation(len(states))
    rc, ln, nd = B.solve_mixed_raw([states[k] for k in order])
    assert rc == want[order][0] and (ln == -1).all() and not nd.any()


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097])
def test_host_buffers_around_the_pinned_size(opts, n):
    """Host-buffer calls pass up to 4096 instances through pinned memory and
    copy larger batches: easy states against the oracle, one invalid among
    them, and a second, smaller call on the same buffers."""
    from oracle import oracle
    from paper_1705_02843_amd import instances as I
    B = opts
    set_mode(B, "batched")
    rng = np.random.Generator(np.random.PCG64(n))
    base = np.stack([I.random_walk(rng, 4, k % 17)[0] for k in range(64)])
    states = base[np.arange(n) % 64].copy()
    want = oracle.solve(base, 4, nthreads=8)
    if n > 1:
        states[n // 2, 0] = states[n // 2, 1]
    for m in (n, (n + 1) // 2):
        rc, ln, nd = B.solve_raw(states[:m])
        k = np.arange(m)
        ok = np.ones(m, bool)
        if n > 1 and n // 2 < m:
            ok[n // 2] = False
        assert rc == (B.OK if ok.all() else B.EINVAL)
        assert (ln[ok] == want.length[k[ok] % 64]).all() and (nd[ok] == want.nodes[k[ok] % 64]).all()
        assert (ln[~ok] == -1).all() and not nd[~ok].any()
