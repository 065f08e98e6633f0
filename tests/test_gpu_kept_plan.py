"""The launch plan that a state keeps from step to step takes up each step's hyper-parameters: against fresh states that
continue from the same point, bit for bit, on every kind of launch."""
import dataclasses

import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl

pytestmark = pytest.mark.gpu

LISTS = {
    "a chain of both precisions": ([(200, 300), (300, 200), (64, 200), (5, 64)], 0),
    "a workgroup each, large tiles, merged products": ([(256, 512)] * 120 + [(1024, 1024)] * 16 + [(300, 700)] * 2, 0),
    "fp32 products": ([(512, 640)] * 6 + [(40, 128)] * 100, 1),
    "chunks of iterations": ([(1536, 4096), (1024, 2048)], 0),
}
# what a schedule changes between steps, and what experiments do
CHANGES = [{}, {"lr": 0.7e-3}, {"weight_decay": 0.3}, {"gamma_coeff": 0.11}, {"ns_a": 3.0, "ns_b": -3.2, "ns_c": 1.3}, {"ns_steps": 3},
           {"momentum": 0.5, "beta_a": 0.5, "alpha": 0.1}, {"lr": 2e-2, "ns_eps": 1e-3}]


@pytest.mark.parametrize("name", LISTS)
def test_hyper_parameters_that_change_from_step_to_step(name):
    shapes, precision = LISTS[name]
    print(f"[case] {name}", flush=True)
    dev = "cuda:0"
    weights = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
    opt = B.MonaOptimizer(weights, ns_precision=precision)
    hp = wl.HParams()
    for k, change in enumerate(CHANGES):
        hp = dataclasses.replace(hp, **change)
        grads = [wl.GradientStream(s, 400 + 1000 * k + i, dev).next() for i, s in enumerate(shapes)]
        copies = [w.clone() for w in weights]
        fresh = B.MonaOptimizer(copies, ns_precision=precision)
        fresh.import_state(opt.export_state(), k)
        opt.step(grads, hp)
        fresh.step(grads, hp)
        torch.cuda.synchronize()
        for i, (w, c) in enumerate(zip(weights, copies)):
            assert torch.equal(w, c), (name, k, i)
