"""Chains of small products as one launch (ns_chain_kernel) at the sizes where they can go wrong: against the float64 oracle,
against the same products launched one by one, and replayed from a HIP graph."""
import ctypes

import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

# (shapes, ns_precision, chain launches)
CASES = {
    # tiles of 32 and one row or column more, wide and tall, K of one slab a wavefront to twelve
    "edges of 32": ([(96, 97), (97, 96), (129, 161), (225, 225), (1500, 70), (66, 1500)], 0, 1),
    "edges of 32, fp32": ([(1, 1), (31, 33), (33, 31), (64, 96), (32, 32), (97, 65), (40, 1300)], 1, 1),
    # positions of 64 x 64 tiles: 256 of 32 x 32 (16 a side) and one row more, and the widest position a chain takes
    "512 and 513 rows": ([(512, 520)], 0, 1),
    "513 rows": ([(513, 520)], 0, 1),
    "seven tiles by eight, four times": ([(400, 500)] * 4, 0, 1),
    # more groups than one chain takes; both precisions in one chain
    "nine groups": ([(70 + 13 * i, 90 + 40 * i) for i in range(9)], 0, 2),
    "both precisions": ([(200, 300), (300, 200), (64, 200), (5, 64), (100, 1)], 0, 1),
}


def steps(shapes, precision, level, count=2):
    weights = [wl.draw_weight(s, 300 + i, torch.float32, "cuda:0") for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer(weights, ns_precision=precision)
    opt.set_profiling(level)
    for k in range(count):
        opt.step([wl.GradientStream(s, 400 + 50 * k + i, "cuda:0").next() for i, s in enumerate(shapes)], wl.HParams())
    torch.cuda.synchronize()
    return weights


@pytest.mark.parametrize("name", CASES)
def test_chains(name):
    shapes, precision, chains = CASES[name]
    print(f"[case] {name}", flush=True)
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    assert B.MonaOptimizer([w.cuda() for w in weights], ns_precision=precision).plan_info(5)["ns_launches"] == chains
    grads = [[wl.GradientStream(s, 400 + 50 * k + i).next() for i, s in enumerate(shapes)] for k in range(2)]
    watch = range(len(shapes))
    opt, dev_w, hist = H.run_gpu(weights, grads, wl.HParams(), precision, watch=watch)
    tol = H.TOL_NS_F32 if precision else H.TOL_NS_BF16
    H.check_history(weights, grads, wl.HParams(), hist, watch, tol, label=name)
    # one by one the products have the same tiles and the same order of sums: the same bits
    for i, (x, y) in enumerate(zip(steps(shapes, precision, 0), steps(shapes, precision, 2))):
        assert torch.equal(x, y), (name, i)


def test_chains_replayed_from_a_graph():
    """The rolls and flags of a chain are cleared by the step's own kernels, so every replay starts from zero."""
    shapes, precision, _ = CASES["nine groups"]
    print("[case] replays", flush=True)
    dev = "cuda:0"
    hp = wl.HParams()
    eager = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
    graph_w = [w.clone() for w in eager]
    opt_e, opt_g = B.MonaOptimizer(eager), B.MonaOptimizer(graph_w)
    grads = [wl.GradientStream(s, 500 + i, dev).next() for i, s in enumerate(shapes)]
    for opt in (opt_e, opt_g):
        opt.step(grads, hp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        opt_g.step(grads, hp)
    for k in range(4):
        for i, g in enumerate(grads):
            g.copy_(wl.GradientStream(g.shape, 600 + 20 * k + i, dev).next())
        opt_e.step(grads, hp)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i in range(len(shapes)):
            assert torch.equal(eager[i], graph_w[i]), (k, i)


def polls(opt, roll, wait):
    return opt.lib.mona_internal_chain_polls(ctypes.c_void_p(opt.state), roll, wait)


@pytest.mark.parametrize("name", CASES)
def test_chains_begun_without_some(name):
    """A roll that is closed at once: those that come later draw their tasks, and the results are the same bits."""
    shapes, precision, _ = CASES[name]
    print(f"[case] {name}", flush=True)
    dev = "cuda:0"
    weights = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer(weights, ns_precision=precision)
    assert polls(opt, 0, 1 << 20) == B.MONA_OK
    for k in range(2):
        opt.step([wl.GradientStream(s, 400 + 50 * k + i, dev).next() for i, s in enumerate(shapes)], wl.HParams())
    assert opt.status() == [0] * len(shapes)
    for i, (x, y) in enumerate(zip(weights, steps(shapes, precision, 0))):
        assert torch.equal(x, y), (name, i)


def test_chains_beside_another_stream():
    """Kernels of another stream hold the CUs for some hundred us at a time, so chains begin with those that are free."""
    print("[case] beside", flush=True)
    shapes, precision, _ = CASES["seven tiles by eight, four times"]
    dev = "cuda:0"
    big = [wl.draw_weight((2048, 1024), 700 + i, torch.float32, dev) for i in range(32)]
    big_g = [wl.GradientStream((2048, 1024), 800 + i, dev).next() for i in range(32)]
    grads = [[wl.GradientStream(s, 400 + 50 * k + i, dev).next() for i, s in enumerate(shapes)] for k in range(2)]
    ends = []
    for busy in (False, True):
        weights = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
        opt, other = B.MonaOptimizer(weights, ns_precision=precision), B.MonaOptimizer(big)
        torch.cuda.synchronize()
        here, there = torch.cuda.Stream(), torch.cuda.Stream()
        if busy:
            with torch.cuda.stream(there):
                for _ in range(6):
                    other.step(big_g, wl.HParams())
        with torch.cuda.stream(here):
            for k in range(20):
                opt.step(grads[k % 2], wl.HParams())
            assert opt.status() == [0] * len(shapes)
        torch.cuda.synchronize()
        ends.append(weights)
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), i


def test_a_wait_that_does_not_end():
    """Chains whose waits may not poll at all: the launch ends, no parameter is touched, the status says so; the next step is whole."""
    shapes, precision, _ = CASES["nine groups"]
    print("[case] no polls", flush=True)
    dev = "cuda:0"
    weights = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
    plain = [w.clone() for w in weights]
    opt, ref = B.MonaOptimizer(weights), B.MonaOptimizer(plain)
    grads = [[wl.GradientStream(s, 500 + 20 * k + i, dev).next() for i, s in enumerate(shapes)] for k in range(2)]
    before = [w.clone() for w in weights]
    assert polls(opt, 64, 0) == B.MONA_OK
    opt.step(grads[0], wl.HParams())
    assert all(s & B.MONA_STATUS_INCOMPLETE for s in opt.status())
    for i in range(len(shapes)):
        assert torch.equal(weights[i], before[i]), i
    assert polls(opt, 64, 1 << 20) == B.MONA_OK
    ref.step(grads[0], wl.HParams())
    for w, p in zip(weights, plain):
        w.copy_(p)                   # (the state arrays are those of a whole step)
    opt.step(grads[1], wl.HParams())
    ref.step(grads[1], wl.HParams())
    assert opt.status() == [0] * len(shapes)
    for i in range(len(shapes)):
        assert torch.equal(weights[i], plain[i]), i
