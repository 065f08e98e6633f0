"""The kernel that takes a whole matrix through all its iterations in one workgroup (ns_matrix_kernel) against the float64
oracle: both short sides, wide and tall, panels that stay in LDS and panels that do not, remainders, odd and even T."""
import dataclasses

import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

COUNT = 120
# (shapes, iterations): every shape COUNT times (as many as make the kernel the better choice at both short sides)
CASES = {
    "p 128, one panel": ([(100, 128)], 5),
    "p 128, tall, two panels and a remainder": ([(300, 97)], 5),
    "p 128, four panels": ([(128, 512), (512, 128)], 5),
    "p 128, five panels": ([(120, 600), (640, 66)], 5),
    "p 256, two panels": ([(256, 256), (200, 256)], 5),
    "p 256, odd sides": ([(131, 389), (643, 255)], 5),
    "p 256, six panels": ([(256, 768), (768, 256)], 5),
    "one iteration": ([(100, 200), (600, 120), (200, 300), (400, 250)], 1),
    "two iterations": ([(100, 200), (600, 120), (200, 300), (400, 250)], 2),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("param", [torch.float32, torch.bfloat16])
def test_matrix_kernel_against_the_oracle(name, param):
    kinds, steps = CASES[name]
    print(f"[case] {name}", flush=True)
    shapes = [s for s in kinds for _ in range(COUNT)]
    watch = [i * COUNT + k for i in range(len(kinds)) for k in (0, COUNT - 1)]
    weights = [wl.draw_weight(s, 300 + i, param) for i, s in enumerate(shapes)]
    hp = wl.HParams(ns_steps=steps)
    assert B.MonaOptimizer([w.cuda() for w in weights]).plan_info(steps)["ns_launches"] == 1
    grads = [[wl.GradientStream(s, 400 + 500 * k + i).next() for i, s in enumerate(shapes)] for k in range(2)]
    opt, dev_w, hist = H.run_gpu(weights, grads, hp, 0, watch=watch)
    if param == torch.float32:
        H.check_history(weights, grads, hp, hist, watch, H.TOL_NS_BF16, label=name)
        return
    ref = H.run_oracle_for(weights, grads, hp, watch)
    for k in range(2):
        for i in watch:
            assert H.rel_fro(hist[k][i].O, ref[i][k]["O"]) <= H.TOL_NS_BF16, (name, k, i)


def test_zero_and_infinite_matrices_among_others():
    """A matrix without gradients has O = 0 and decays; one with an infinite gradient keeps its parameter; the others go on."""
    print("[case] zero, infinite", flush=True)
    shapes = [(130, 300)] * COUNT
    weights = [wl.draw_weight(s, 300 + i, torch.float32, "cuda:0") for i, s in enumerate(shapes)]
    grads = [wl.GradientStream(s, 400 + i, "cuda:0").next() for i, s in enumerate(shapes)]
    grads[3].zero_()
    grads[5][7, 11] = float("inf")
    before = [w.clone() for w in weights]
    plain = [w.clone() for w in weights]
    hp = wl.HParams()
    opt = B.MonaOptimizer(weights)
    opt.step(grads, hp)
    assert opt.status()[3] == 1 and opt.status()[5] & 2
    assert torch.allclose(weights[3], before[3] * (1.0 - hp.lr * hp.weight_decay), rtol=1e-6, atol=0.0)
    assert torch.equal(weights[5], before[5])
    alone = B.MonaOptimizer(plain)
    alone.step([g if i not in (3, 5) else torch.ones_like(g) for i, g in enumerate(grads)], dataclasses.replace(hp))
    for i in range(COUNT):
        if i not in (3, 5):
            assert torch.equal(weights[i], plain[i]), i


@pytest.mark.parametrize("shape", [(256, 768), (768, 256)])
@pytest.mark.parametrize("param", [torch.float32, torch.bfloat16])
def test_the_bits_of_the_large_tile_kernel(shape, param):
    """A short side of 256: every sum runs over K in the order of the large-tile kernel and is rounded in the same places (the
    scale of the first iteration behind the sum of the apply), so the parameters are the same, bit for bit.  The large
    tiles: the same matrices, fewer of them, beside matrices that fill the chip with such tiles."""
    print(f"[case] {shape}", flush=True)
    few, dev = 36, "cuda:0"

    def run(shapes, level):
        weights = [wl.draw_weight(s, 300 + i, param, dev) for i, s in enumerate(shapes)]
        opt = B.MonaOptimizer(weights)
        opt.set_profiling(level)
        for k in range(2):
            opt.step([wl.GradientStream(s, 400 + 1000 * k + i, dev).next() for i, s in enumerate(shapes)], wl.HParams())
        torch.cuda.synchronize()
        return opt, weights

    beside = [shape] * few + [(1024, 1024)] * 16
    opt, _ = run(beside, 2)
    assert {r["tile"] for r in opt.last_step_launches()} == {256256}
    alone = B.MonaOptimizer([wl.draw_weight(shape, i, param, dev) for i in range(COUNT)])
    assert alone.plan_info(5)["ns_launches"] == 1
    want, got = run(beside, 0)[1], run([shape] * COUNT, 0)[1]
    for i in range(few):
        assert torch.equal(want[i], got[i]), i


@pytest.mark.parametrize("shapes", [[(768, 256)] * 128 + [(256, 768)] * 128 + [(100, 300)] * 80,
                                    [(256, 512)] * COUNT + [(2048, 2048)] * 8 + [(100, 100)] * 200 + [(30, 500)] * 3])
def test_groups_timed_one_by_one_give_the_same_bits(shapes):
    """Profiling level 2 launches and times the groups of the kernel one by one, and the step's results stay what they are."""
    print(f"[case] {len(shapes)} matrices", flush=True)
    ends = []
    for level in (0, 2):
        weights = [wl.draw_weight(s, 300 + i, torch.bfloat16, "cuda:0") for i, s in enumerate(shapes)]
        opt = B.MonaOptimizer(weights)
        opt.set_profiling(level)
        for k in range(2):
            opt.step([wl.GradientStream(s, 400 + 1000 * k + i, "cuda:0").next() for i, s in enumerate(shapes)], wl.HParams())
        torch.cuda.synchronize()
        ends.append(weights)
    records = opt.last_step_launches()
    whole = [(r["m"], r["n"]) for r in records if r["kind"] == 4]
    assert len(whole) == len(set(whole)) and set(whole) >= {s for s in shapes if max(s) < 800 and min(s) > 64}
    assert all(r["ms"] > 0 and r["flops"] > 0 for r in records)
    flops = opt.plan_info(5)["ns_flops_issued"]
    assert abs(sum(r["flops"] for r in records) - flops) <= 1e-9 * flops
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), i


def test_matrix_kernel_beside_other_groups():
    """Matrices with a workgroup each beside large tiles, merged small products of both precisions and a long chain of K."""
    kinds = [(256, 512, COUNT), (1024, 1024, 16), (100, 100, 200), (30, 500, 3), (300, 700, 2), (120, 600, 150)]
    print("[case] beside", flush=True)
    shapes = [(m, n) for m, n, c in kinds for _ in range(c)]
    firsts = [sum(c for _, _, c in kinds[:i]) for i in range(len(kinds))]
    watch = [f + k for f, (_, _, c) in zip(firsts, kinds) for k in (0, c - 1)]
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer([w.cuda() for w in weights])
    grads = [[wl.GradientStream(s, 400 + 500 * k + i).next() for i, s in enumerate(shapes)] for k in range(2)]
    opt.set_profiling(2)
    opt.step([g.cuda() for g in grads[0]], wl.HParams())
    records = opt.last_step_launches()
    assert {(r["m"], r["n"]) for r in records if r["kind"] == 4} == {(256, 512), (100, 100), (120, 600)}
    assert 256256 in {r["tile"] for r in records if r["kind"] != 4}
    opt, dev_w, hist = H.run_gpu(weights, grads, wl.HParams(), 0, watch=watch)
    H.check_history(weights, grads, wl.HParams(), hist, watch, H.TOL_NS_BF16, label="beside")
