"""The parameter update in the last product of large and of small tiles, for rows of W of any length (pieces of 8 values that are aligned
like one, the last one of a row partly outside, or rows of whole pieces) and for groups of bf16 parameters, of fp32 ones and of both,
against the update formed from the stored O in float64."""
import ctypes

import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

# (shape, how many, schedule, tile of the last product): large tiles in the literal and in a fused schedule, tall and wide; 128 x 128 and
# 64 x 64 tiles, in launches and in a chain; the kernel that takes a matrix through all of its iterations (one record, kind 4)
CASES = {
    "large tiles, literal": ((505, 509), 44, B.MONA_NS_SCHEDULE_LITERAL, 256256),
    "large tiles, tall": ((1022, 510), 20, B.MONA_NS_SCHEDULE_FUSED, 256256),
    "large tiles, wide": ((510, 1023), 20, B.MONA_NS_SCHEDULE_FUSED, 256256),
    "large tiles, literal, rows of whole pieces": ((505, 504), 44, B.MONA_NS_SCHEDULE_LITERAL, 256256),
    "large tiles, tall, rows of whole pieces": ((1022, 504), 20, B.MONA_NS_SCHEDULE_FUSED, 256256),
    "large tiles, wide, rows of whole pieces": ((510, 1016), 20, B.MONA_NS_SCHEDULE_FUSED, 256256),
    "tiles of 128": ((500, 613), 13, B.MONA_NS_SCHEDULE_AUTO, 128128),
    "tiles of 128, a side just past three": ((385, 1007), 6, B.MONA_NS_SCHEDULE_AUTO, 128128),
    "tiles of 64": ((385, 1007), 3, B.MONA_NS_SCHEDULE_AUTO, 64064),
    "a chain": ((297, 131), 2, B.MONA_NS_SCHEDULE_AUTO, 32032),
    "a chain, tiles of 64": ((331, 509), 3, B.MONA_NS_SCHEDULE_AUTO, 64064),
    "a workgroup to a matrix": ((97, 131), 2, B.MONA_NS_SCHEDULE_AUTO, 128128),
}


@pytest.mark.parametrize("of", ["fp32", "bf16", "both"])
@pytest.mark.parametrize("name", CASES)
def test_update_of_rows_of_any_length(name, of):
    shape, count, schedule, tile = CASES[name]
    print(f"[case] {name}, {of}", flush=True)
    kinds = [torch.bfloat16 if of == "bf16" or (of == "both" and i % 2) else torch.float32 for i in range(count)]
    weights = [wl.draw_weight(shape, 300 + i, kinds[i]) for i in range(count)]
    grads = [[wl.GradientStream(shape, 500 + i).next() for i in range(count)]]
    watch = (0, 1, count - 2, count - 1)
    hp = wl.HParams()
    opt, _, hist = H.run_gpu(weights, grads, hp, 0, watch=watch, ns_schedule=schedule)
    for i in watch:
        s = hist[0][i]
        want = H.expected_update(s.W_before, s.O, hp, False)
        terms = abs(s.W_before) + abs(want - s.W_before)
        # half an ulp for the store and three fp32 roundings of the terms
        ulp = 2.0 ** -8 if kinds[i] == torch.bfloat16 else 2.0 ** -23
        assert (abs(s.W - want) <= abs(want) * ulp + terms * 2.0 ** -22).all(), i
    assert (opt.lib.mona_internal_chain_kind(ctypes.c_void_p(opt.state)) >= 0) == name.startswith("a chain")
    opt.set_profiling(2)                         # (timed one by one, products keep their tiles)
    opt.step([g.cuda() for g in grads[0]], hp)
    last = opt.last_step_launches()[-1]
    assert last["tile"] == tile and (last["kind"] == 4) == (name == "a workgroup to a matrix")
