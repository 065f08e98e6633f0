"""The small-tile product kernels (64 x 64 and 128 x 128, one launch for several shape groups) at the sizes where they can
go wrong, against the float64 oracle."""
import dataclasses
import itertools

import numpy as np
import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

# (shapes, ns_precision, matrices to check)
CASES = {
    # (so few tiles go out as chains, see test_gpu_chains.py; "more of them" below are launches of their own)
    # a tile and one more row or column, short and long K (one to eleven slabs a wavefront), wide and tall
    "edges of 64": ([(65, 65), (128, 129), (129, 128), (192, 1300), (1300, 192), (66, 2700)], 0, range(6)),
    # more groups than one launch takes, of unequal sizes
    "eleven groups": ([(70 + 13 * i, 90 + 40 * ((7 * i) % 11)) for i in range(11)], 0, range(11)),
    # enough 128 x 128 tiles, at most one a CU (13 x 10) and more (13 x 20), last tile partly padding
    "tiles of 128": ([(500, 610)] * 13 + [(610, 500)] * 2, 0, (0, 12, 13, 14)),
    # matrices with a workgroup each, around the count from which a single tile each is large under a forced schedule
    "111 large tiles": ([(256, 512)] * 111, 0, (0, 110)),
    "112 large tiles": ([(256, 512)] * 112, 0, (0, 111)),
    # the most tiles of 256 x 256 that a product has on small tiles, and the fewest that it has on large ones
    "126 large tiles": ([(500, 510)] * 42, 0, (0, 41)),
    "129 large tiles": ([(500, 510)] * 43, 0, (0, 42)),
    # groups that fill half the chip run apart, the smaller ones share their launches, in either precision
    "apart and merged": ([(520, 640)] * 9 + [(640, 700)] * 3 + [(300, 260)] * 4 + [(70, 5)], 0, (0, 9, 12, 16)),
    "apart and merged, fp32": ([(520, 640)] * 9 + [(640, 700)] * 3 + [(300, 260)] * 4 + [(70, 5)], 1, (0, 9, 12, 16)),
    # the most matrices whose pointers travel with a launch, and one more: three steps, each with new gradient buffers
    "96 matrices": ([(40, 72)] * 96, 0, (0, 95)),
    "97 matrices": ([(40, 72)] * 97, 0, (0, 96)),
    # fp32 products: 64 x 64 tiles with and without company on the CU, 128 x 128 tiles for the last product
    "fp32 edges": ([(3, 5), (64, 64), (65, 200), (200, 65), (130, 1030)], 1, range(5)),
    "fp32 tiles of 128": ([(700, 1100)] * 10 + [(1100, 700)], 1, (0, 9, 10)),
}


# Too many tiles for a chain, too few matrices for a workgroup each: (shapes, ns_precision, matrices to check, launches, tiles)
MORE = {
    "edges of 64, more of them": ([s for s in CASES["edges of 64"][0] for _ in range(6)], 0, range(0, 36, 6), 15, {64064, 128128}),
    "eleven groups, more of them": ([s for s in CASES["eleven groups"][0] for _ in range(8)], 0, range(0, 88, 8), 30, {64064, 128128}),
    "edges of 128": ([(129, 1100)] * 16 + [(1100, 257)] * 10, 0, (0, 15, 16, 25), 15, {64064, 128128}),
    "fp32 edges, more of them": ([s for s in CASES["fp32 edges"][0] for _ in range(40)], 1, range(0, 200, 40), 45, {64064}),
}


@pytest.mark.parametrize("name", MORE)
def test_launches_of_small_products_against_the_oracle(name):
    shapes, precision, watch, launches, tiles = MORE[name]
    print(f"[case] {name}", flush=True)
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer([w.cuda() for w in weights], ns_precision=precision)
    assert opt.plan_info(5)["ns_launches"] == launches
    grads = [[wl.GradientStream(s, 400 + i).next() for i, s in enumerate(shapes)]]
    opt.set_profiling(2)
    opt.step([g.cuda() for g in grads[0]], wl.HParams())
    assert {r["tile"] for r in opt.last_step_launches()} == tiles
    opt, dev_w, hist = H.run_gpu(weights, grads, wl.HParams(), precision, watch=watch)
    H.check_history(weights, grads, wl.HParams(), hist, watch, H.TOL_NS_F32 if precision else H.TOL_NS_BF16, label=name)


@pytest.mark.parametrize("count, tiles", [(111, {128128}), (112, {256256})])
def test_single_large_tiles_under_a_forced_schedule(count, tiles):
    """p x p products of a single large tile: on small tiles up to 111 matrices, on large ones from 112 on (the pairwise schedule:
    literal iterations of so many take the kernel with a workgroup for each matrix)."""
    print(f"[case] {count}", flush=True)
    shapes, watch = [(256, 512)] * count, (0, count - 1)
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer([w.cuda() for w in weights], ns_schedule=B.MONA_NS_SCHEDULE_PAIRS)
    grads = [[wl.GradientStream(s, 400 + i).next() for i, s in enumerate(shapes)]]
    opt.set_profiling(2)
    opt.step([g.cuda() for g in grads[0]], wl.HParams())
    assert {r["tile"] for r in opt.last_step_launches() if r["kind"] != 2} == tiles
    opt, dev_w, hist = H.run_gpu(weights, grads, wl.HParams(), 0, watch=watch, ns_schedule=B.MONA_NS_SCHEDULE_PAIRS)
    H.check_history(weights, grads, wl.HParams(), hist, watch, H.TOL_NS_BF16, label=str(count))


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("param", [torch.float32, torch.bfloat16])
def test_small_products_against_the_oracle(name, param):
    shapes, precision, watch = CASES[name]
    print(f"[case] {name}", flush=True)
    weights = [wl.draw_weight(s, 300 + i, param) for i, s in enumerate(shapes)]
    streams = [wl.GradientStream(s, 400 + i) for i, s in enumerate(shapes)]
    grads = [[g.next() for g in streams] for _ in range(3 if name.endswith("matrices") else 1)]
    hp = wl.HParams()
    opt, dev_w, hist = H.run_gpu(weights, grads, hp, precision, watch=watch)
    # the suite's bounds: bf16 products round every stored intermediate to 8 bits (measured 1.1e-2 to 1.4e-2 on short
    # sides of 64 and more), fp32 products are right to a few 1e-6
    tol = H.TOL_NS_F32 if precision else H.TOL_NS_BF16
    if param == torch.float32:
        H.check_history(weights, grads, hp, hist, watch, tol, label=name)
        return
    # bf16 parameters: O against the oracle, and the stored parameter against the update formed from that O in float64:
    # half an ulp for the store, and three fp32 roundings of the terms (which cancel where the result is tiny)
    ref = H.run_oracle_for(weights, grads, hp, watch)
    for k, i in itertools.product(range(len(grads)), watch):
        s = hist[k][i]
        assert H.rel_fro(s.O, ref[i][k]["O"]) <= tol, (name, k, i)
        want = H.expected_update(s.W_before, s.O, hp, False)
        terms = np.abs(s.W_before) + np.abs(want - s.W_before)
        assert (np.abs(s.W - want) <= np.abs(want) * 2.0 ** -8 + terms * 2.0 ** -22).all(), (name, k, i)


@pytest.mark.parametrize("name", ["edges of 64", "apart and merged", "apart and merged, fp32"])
def test_launches_timed_one_by_one_give_the_same_bits(name):
    shapes, precision, _ = CASES[name]
    shapes = shapes + [(500, 610), (640, 500), (512, 700)]
    print(f"[case] {name}", flush=True)
    ends = []
    for level in (0, 2):
        weights = [wl.draw_weight(s, 300 + i, torch.float32, "cuda:0") for i, s in enumerate(shapes)]
        opt = B.MonaOptimizer(weights, ns_precision=precision)
        opt.set_profiling(level)
        for k in range(2):
            opt.step([wl.GradientStream(s, 400 + 50 * k + i, "cuda:0").next() for i, s in enumerate(shapes)], wl.HParams())
        torch.cuda.synchronize()
        ends.append(weights)
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), (name, i)


def test_padding_stays_zero_when_the_iterations_change_from_step_to_step():
    """The tile of a product depends on what shares its launch, and that on the number of iterations: 1080 x 6000 (17 tiles of
    64 a side, or 9 of 128 with 64 columns of padding) has another tile at some positions of a chain of 3, 5 and 9 iterations,
    so a buffer's padding may be written by one step and read, unwritten, by the next.  Powers of a in it would leave the bf16
    range within 75 steps and turn the parameter into NaN; O must be that of the same gradients in a fresh state, bit for bit."""
    print("[case] iterations 9, then 5 and 3 in turn", flush=True)
    shapes = [(1080, 6000), (1024, 1536), (1000, 1000)]
    dev = "cuda:0"
    hp = dataclasses.replace(wl.HParams(), flags=B.MONA_FLAG_KEEP_O)
    grads = [wl.GradientStream(s, 700 + i, dev).next() for i, s in enumerate(shapes)]
    weights = [wl.draw_weight(s, 600 + i, torch.float32, dev) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer(weights)
    for k, steps in enumerate([9] + [5, 3] * 40):
        opt.step(grads, dataclasses.replace(hp, ns_steps=steps))
        if k % 20 == 0:
            torch.cuda.synchronize()
            print(f"[step] {k}", flush=True)
    saved = opt.export_state()
    opt.step(grads, hp)
    got = [opt.last_o(i).clone() for i in range(len(shapes))]
    fresh = B.MonaOptimizer(weights)
    fresh.import_state(saved, 1)
    fresh.step(grads, hp)
    for i in range(len(shapes)):
        assert torch.isfinite(weights[i]).all(), i
        assert torch.equal(got[i], fresh.last_o(i)), i
