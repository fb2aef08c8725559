"""The work that programs built on this library have it do, as timed cases.

Every case is one pass through a public entry point of
``paper_1705_02843_amd.bpida`` on seeded sliding-tile states, with the options
a program would run it with: the library's defaults, or the autotuner's table
applied as the benchmark does.  Inputs are non-backtracking random blank walks
from the goal, drawn for a whole batch at a time.

    walk40    end states of 40-move walks (easy: about 1.5e5 nodes each)
    md30_38   300-move walks whose end state has Manhattan distance 30..38
              (the stand-in for the paper's 100-instance set)
    uneven    walks of U{20..300} moves, Manhattan distance at most 38: the
              depths of a mixed stream, a few instances holding most nodes
    walk60    60-move walks (the 5x5 part of the mixed workload)
"""
import math
import time

import numpy as np
import torch

from paper_1705_02843_amd import autotune, bpida

OPS_PER_NODE = 64  # integer operations one expanded node cannot do without (bench.py)
# mean expanded nodes of one instance, all limits, from the stored oracle results
MEAN_NODES = {("walk40", 4): 1.5e5, ("md30_38", 4): 2.2e8, ("uneven", 4): 1.4e8,
              ("uneven", 3): 3.7e3, ("walk60", 5): 1.06e8}
DEFAULTS = {"mode": 1, "nodes_per_round": 64, "lds_stack_capacity": -1, "wg_size": 64,
            "frontier_depth": -1, "max_workgroups": 0, "donate_every": 128, "donate_min": -1,
            "queue_chunk": 64}
_applied = None  # the options this process has set last


def listed():
    return [
        # a program that asks for one puzzle at a time, from host memory
        {"name": "one_easy", "entry": "host", "width": 4, "recipe": "walk40", "n": 1, "tuned": False},
        # one hard puzzle alone on the GPU: what its own limits and their spreading cost
        {"name": "one_hard", "entry": "device", "width": 4, "recipe": "md30_38", "n": 1, "tuned": False},
        # a small batch of easy puzzles (a puzzle game's hint server)
        {"name": "batch64_easy", "entry": "device", "width": 4, "recipe": "walk40", "n": 64, "tuned": True},
        # the paper's experiment: 100 hard puzzles
        {"name": "batch100_hard", "entry": "device", "width": 4, "recipe": "md30_38", "n": 100, "tuned": True},
        # the benchmark's batch: 4096 puzzles of very different depth
        {"name": "batch4096", "entry": "device", "width": 4, "recipe": "uneven", "n": 4096, "tuned": True},
        # a ragged batch enqueued on the caller's stream with the library's default options
        {"name": "async777", "entry": "async", "width": 4, "recipe": "uneven", "n": 777, "tuned": False},
        # 8-puzzles: thousands of tiny searches
        {"name": "w3_2048", "entry": "device", "width": 3, "recipe": "uneven", "n": 2048, "tuned": True},
        # 24-puzzles
        {"name": "w5_61", "entry": "device", "width": 5, "recipe": "walk60", "n": 61, "tuned": True},
        # the three widths in one launch, in the mixed workload's proportions
        {"name": "mixed1088", "entry": "mixed", "width": 0, "recipe": "uneven", "n": 1088, "tuned": True},
        # optimal move sequences as well as lengths
        {"name": "paths40", "entry": "paths", "width": 4, "recipe": "md30_38", "n": 40, "tuned": False},
        # Alg. 1 as printed: one launch per instance and limit, statically balanced
        {"name": "plain12", "entry": "plain", "width": 4, "recipe": "md30_38", "n": 12, "tuned": False},
        # a burst of requests to the continuous-batching server
        {"name": "serve200", "entry": "serve", "width": 4, "recipe": "uneven", "n": 200, "tuned": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("batch", "batch", "batch", "w3", "w5", "mixed", "paths", "plain", "serve"))
    if kind == "batch":
        recipe = rng.choice(("walk40", "md30_38", "uneven"))
        top = {"walk40": 4096, "md30_38": 1000, "uneven": 3000}[recipe]
        entry = rng.choice(("host", "device", "async", "noalloc"))
        return {"entry": entry, "width": 4, "recipe": recipe, "n": _log_int(rng, 1, top),
                "tuned": rng.random() < 0.5}
    if kind == "w3":
        return {"entry": rng.choice(("host", "device", "async")), "width": 3, "recipe": "uneven",
                "n": _log_int(rng, 1, 8192), "tuned": rng.random() < 0.5}
    if kind == "w5":
        return {"entry": "device", "width": 5, "recipe": "walk60", "n": _log_int(rng, 8, 200),
                "tuned": rng.random() < 0.5}
    if kind == "mixed":
        return {"entry": "mixed", "width": 0, "recipe": "uneven", "n": _log_int(rng, 17, 3000),
                "tuned": rng.random() < 0.5}
    if kind == "paths":
        recipe = rng.choice(("walk40", "md30_38"))
        return {"entry": "paths", "width": 4, "recipe": recipe, "n": _log_int(rng, 1, 80), "tuned": False}
    if kind == "plain":
        recipe = rng.choice(("walk40", "md30_38"))
        return {"entry": "plain", "width": 4, "recipe": recipe, "n": _log_int(rng, 1, 24), "tuned": False}
    return {"entry": "serve", "width": 4, "recipe": rng.choice(("walk40", "uneven")),
            "n": _log_int(rng, 8, 500), "tuned": False}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _walks(rng, width, lengths):
    """End states of non-backtracking blank walks from the goal, one per entry of lengths."""
    n = lengths.shape[0]
    cells = width * width
    s = np.tile(np.arange(cells, dtype=np.uint8), (n, 1))
    blank = np.zeros(n, np.int64)
    prev = np.full(n, -1)
    step = np.array([-width, -1, 1, width])
    cell = np.arange(cells)
    legal = np.stack([cell >= width, cell % width > 0, cell % width < width - 1,
                      cell < cells - width], axis=1)
    rows = np.arange(n)
    for k in range(int(lengths.max()) if n else 0):
        ok = legal[blank]
        undo = prev >= 0
        ok[rows[undo], 3 - prev[undo]] = False
        pick = (rng.random(n) * ok.sum(axis=1)).astype(np.int64)
        a = (np.cumsum(ok, axis=1) > pick[:, None]).argmax(axis=1)
        go = k < lengths
        to = np.where(go, blank + step[a], blank)
        moved = s[rows, to]
        s[rows, to] = np.where(go, 0, moved)
        s[rows[go], blank[go]] = moved[go]
        blank = to
        prev = np.where(go, a, prev)
    return s


def _manhattan(s, width):
    cell = np.arange(width * width)
    t = s.astype(np.int64)
    d = np.abs(cell // width - t // width) + np.abs(cell % width - t % width)
    return np.where(t == 0, 0, d).sum(axis=1)


def _states(rng, recipe, width, n):
    if recipe == "walk40":
        return _walks(rng, width, np.full(n, 40))
    if recipe == "walk60":
        return _walks(rng, width, np.full(n, 60))
    lo, hi = (30, 38) if recipe == "md30_38" else (0, 38 if width == 4 else 999)
    got = np.zeros((0, width * width), np.uint8)
    while got.shape[0] < n:
        m = 2 * (n - got.shape[0]) + 16
        lengths = np.full(m, 300) if recipe == "md30_38" else rng.integers(20, 301, size=m)
        s = _walks(rng, width, lengths)
        md = _manhattan(s, width)
        got = np.concatenate([got, s[(md >= lo) & (md <= hi)]])
    return np.ascontiguousarray(got[:n])


def _mixed_counts(n):
    # the mixed workload's proportions: 8 3x3 and 8 4x4 to one 5x5
    n5 = n // 17
    n3 = (n - n5) // 2
    return n3, n - n5 - n3, n5


def _draw_inputs(case, seed):
    """[(width, states)] in the order they are handed over."""
    rng = np.random.default_rng([seed, case["n"], case["width"]])
    if case["entry"] == "mixed":
        n3, n4, n5 = _mixed_counts(case["n"])
        return [(3, _states(rng, "uneven", 3, n3)), (4, _states(rng, "uneven", 4, n4)),
                (5, _states(rng, "walk60", 5, n5))]
    return [(case["width"], _states(rng, case["recipe"], case["width"], case["n"]))]


def _options(case):
    opts = dict(DEFAULTS)
    if case["entry"] == "plain":
        opts["mode"] = 0
    elif case["tuned"]:
        opts.update(autotune.lookup(case["n"], case["width"]) or {})
    return opts


def prepare(case, seed):
    parts = _draw_inputs(case, seed)
    st = {"entry": case["entry"], "width": case["width"], "options": _options(case)}
    n = sum(s.shape[0] for _, s in parts)
    if case["entry"] in ("host", "serve"):
        st["states"] = parts[0][1]
        return st
    flat = np.concatenate([s.reshape(-1) for _, s in parts])
    if case["entry"] == "mixed":
        st["widths"] = np.concatenate([np.full(s.shape[0], w, np.int32) for w, s in parts])
        st["states"] = torch.from_numpy(flat).cuda()
    else:
        st["states"] = torch.from_numpy(flat.reshape(n, -1)).cuda()
    st["len"] = torch.empty(n, dtype=torch.int32, device="cuda")
    st["nodes"] = torch.empty((n, bpida.MAX_THRESHOLDS), dtype=torch.int64, device="cuda")
    if case["entry"] == "paths":
        st["path"] = torch.empty((n, bpida.MAX_PATH), dtype=torch.uint8, device="cuda")
    if case["entry"] in ("async", "noalloc"):
        st["status"] = torch.empty(n, dtype=torch.int32, device="cuda")
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def _use(options):
    """Sets the library's options where they differ from the ones set last."""
    global _applied
    if _applied != options:
        for k, v in options.items():
            bpida.set_option(k, v)
        _applied = dict(options)


def _checked(rc):
    if rc != bpida.OK:
        raise bpida.BpidaError(rc, "solve")


def _serve(states):
    n = states.shape[0]
    length = np.empty(n, np.int32)
    nodes = np.empty((n, bpida.MAX_THRESHOLDS), np.uint64)
    status = np.empty(n, np.int32)
    with bpida.Server(max_inflight=512, ring_capacity=1024) as srv:
        pending = {srv.submit(states[i]): i for i in range(n)}
        while pending:
            for t in list(pending):
                r = srv.poll(t)
                if r is not None:
                    i = pending.pop(t)
                    length[i], nodes[i], status[i] = r
            time.sleep(0)
    return {"len": length, "nodes": nodes.view(np.int64), "status": status}


def run(st):
    _use(st["options"])
    entry, width = st["entry"], st["width"]
    if entry == "host":
        rc, length, nodes = bpida.solve_raw(st["states"], width)
        _checked(rc)
        return {"len": length, "nodes": nodes.view(np.int64)}
    if entry == "serve":
        return _serve(st["states"])
    out = {"len": st["len"], "nodes": st["nodes"]}
    if entry == "async" or entry == "noalloc":
        call = bpida.solve_device_async if entry == "async" else bpida.solve_device_noalloc
        _checked(call(st["states"], st["len"], st["nodes"], st["status"], width=width))
        return dict(out, status=st["status"])
    if entry == "mixed":
        _checked(bpida.solve_mixed_device(st["states"], st["widths"], st["len"], st["nodes"]))
        return out
    if entry == "paths":
        _checked(bpida.solve_paths_device(st["states"], st["len"], st["nodes"], st["path"], width=width))
        return dict(out, path=st["path"])
    _checked(bpida.solve_device(st["states"], st["len"], st["nodes"], width=width))
    return out


def work(case):
    """States in; lengths and counts (and paths) out; the nodes every limit expands."""
    parts = [(case["width"], case["recipe"], case["n"])]
    if case["entry"] == "mixed":
        parts = list(zip((3, 4, 5), ("uneven", "uneven", "walk60"), _mixed_counts(case["n"])))
    by = sum(k * (w * w + 4 + 8 * bpida.MAX_THRESHOLDS) for w, _, k in parts)
    if case["entry"] == "paths":
        by += case["n"] * bpida.MAX_PATH
    return {"bytes": by, "flops": OPS_PER_NODE * sum(k * MEAN_NODES[(r, w)] for w, r, k in parts)}


# ---------------------------------------------------------------------------
# The same answers from plain numpy
# ---------------------------------------------------------------------------

def _count(states, width):
    """Optimal lengths and nodes per limit by a level-by-level f-limited
    search of all states at once, one limit after the other."""
    n, cells = states.shape
    length = np.full(n, -1, np.int32)
    nodes = np.zeros((n, 64), np.int64)
    h0 = _manhattan(states, width)
    step = np.array([-width, -1, 1, width])
    cell = np.arange(cells)
    legal = np.stack([cell >= width, cell % width > 0, cell % width < width - 1,
                      cell < cells - width], axis=0)
    goal = np.arange(cells, dtype=np.uint8)
    dist = (np.abs(cell[:, None] // width - cell[None] // width)
            + np.abs(cell[:, None] % width - cell[None] % width))
    dist[0] = 0  # the blank does not count
    for col in range(64):
        inst = np.nonzero(length < 0)[0]
        if inst.size == 0:
            break
        s, slack = states[inst], np.full(inst.size, 2 * col)
        blank, last = (s == 0).argmax(axis=1), np.full(inst.size, -1)
        while inst.size:
            nodes[:, col] += np.bincount(inst, minlength=n)
            at_goal = inst[(s == goal).all(axis=1)]
            length[at_goal] = h0[at_goal] + 2 * col
            nxt = []
            for a in range(4):
                k = np.nonzero(legal[a][blank] & (last != 3 - a))[0]
                b, to = blank[k], blank[k] + step[a]
                t = s[k, to]
                left = slack[k] - 1 - dist[t, b] + dist[t, to]
                k, b, to, t, left = (x[left >= 0] for x in (k, b, to, t, left))
                c = s[k]
                c[np.arange(k.size), to] = 0
                c[np.arange(k.size), b] = t
                nxt.append((inst[k], c, left, to, np.full(k.size, a)))
            inst, s, slack, blank, last = (np.concatenate(x) for x in zip(*nxt))
    return length, nodes


def exact(case, seed):
    """Lengths and counts for the small searches; the others would take minutes."""
    if case["entry"] in ("mixed", "plain", "paths", "serve"):
        return None
    if case["n"] * MEAN_NODES[(case["recipe"], case["width"])] > 2e7:
        return None
    length, nodes = _count(_draw_inputs(case, seed)[0][1], case["width"])
    out = {"len": length, "nodes": nodes}
    if case["entry"] in ("async", "noalloc"):
        out["status"] = np.ones(case["n"], np.int32)
    return out
