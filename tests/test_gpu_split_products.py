"""fp32-class products on the bf16 matrix instructions (ns_small_kernel_split) against the float64 oracle: both tiles, wide
and tall, remainders, and the shortest K that takes that path."""
import numpy as np
import pytest
import torch

from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

CASES = {
    "64 x 64, K of 256": [(130, 200)] * 60,
    "64 x 64, a row more than three tiles": [(193, 700)] * 30 + [(700, 193)] * 8,
    "128 x 128": [(512, 640)] * 14,
    "128 x 128, remainders, tall": [(1030, 300)] * 24,
    "both tiles in turn": [(1024, 1300)] * 3,
    "short K beside long": [(96, 300)] * 100 + [(300, 96)] * 3,
}


@pytest.mark.parametrize("name", CASES)
def test_split_products_against_the_oracle(name):
    shapes = CASES[name]
    print(f"[case] {name}", flush=True)
    watch = (0, len(shapes) - 1)
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    grads = [[wl.GradientStream(s, 400 + 500 * k + i).next() for i, s in enumerate(shapes)] for k in range(2)]
    # a matrix whose entries span fifteen orders of magnitude: the planes of the small ones must not be lost
    for k in range(2):
        g = grads[k][0]
        g *= torch.logspace(0, -15, g.shape[1], dtype=torch.float64).float()
    opt, dev_w, hist = H.run_gpu(weights, grads, wl.HParams(), 1, watch=watch)
    H.check_history(weights, grads, wl.HParams(), hist, watch, H.TOL_NS_F32, label=name)
    # fp32 rounds every product's sum to 2^-24 of it; five iterations of three products that amplify by at most 3.4445 at first
    # leave a few 1e-6, here on the ordinary matrix
    ref = H.run_oracle_for(weights, grads, wl.HParams(), watch)
    for k in range(2):
        assert H.rel_fro(hist[k][watch[1]].O, ref[watch[1]][k]["O"]) <= 5e-6, (name, k)
        assert np.isfinite(hist[k][0].O).all()
