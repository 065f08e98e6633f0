"""The elementwise pass in its forms: rows of any length (groups of 4 elements that straddle rows of the working copy), one launch for what
stands before the products of a small step, and a norm out of range there, against the float64 oracle."""
import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

# (33 matrices are one too many for the one launch)
SHAPES = [(1, 1), (1, 3), (3, 1), (67, 65), (65, 66), (70, 67), (66, 68), (129, 65), (4097, 1), (100, 131)]


@pytest.mark.parametrize("more", [0, 33])
@pytest.mark.parametrize("g_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("state_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("form", ["two_buffer", "one_buffer"])
def test_rows_of_any_length(more, g_dtype, state_dtype, form):
    print(f"[case] {more} {g_dtype} {state_dtype} {form}", flush=True)
    shapes = SHAPES + [(66, 67)] * more
    weights = [wl.draw_weight(s, 300 + i, torch.float32) for i, s in enumerate(shapes)]
    grads = [[wl.GradientStream(s, 400 + 100 * k + i).next().to(g_dtype) for i, s in enumerate(shapes)] for k in range(3)]
    accel = B.MONA_ACCEL_ONE_BUFFER if form == "one_buffer" else B.MONA_ACCEL_TWO_BUFFER
    ends = []
    for level in (0, 2):                          # (profiling level 2 takes the pass, the norms and the pointers as launches of their own)
        dev_w = [w.cuda() for w in weights]
        opt = B.MonaOptimizer(dev_w, state_dtype=state_dtype, g_dtype=g_dtype, accel_form=accel)
        opt.set_profiling(level)
        for g in grads:
            opt.step([x.cuda() for x in g], wl.HParams())
        torch.cuda.synchronize()
        assert opt.status() == [0] * len(shapes)
        ends.append((dev_w, [opt.momentum(i).clone() for i in range(len(shapes))]))
    for i in range(len(shapes)):
        assert torch.equal(ends[0][0][i], ends[1][0][i]) and torch.equal(ends[0][1][i], ends[1][1][i]), i
    # M against Alg. 1 in float64, with the roundings of a bf16 state: half an ulp of A and of G_{k-1} a step, times alpha = -5
    hp = wl.HParams()
    tol = 1e-6 if state_dtype == torch.float32 and form == "two_buffer" else (2e-6 if state_dtype == torch.float32 else 3 * 5 * 2.0 ** -8)
    for i, s in enumerate(shapes):
        a, m, gp = (torch.zeros(s, dtype=torch.float64) for _ in range(3))
        for g in (x[i].double() for x in grads):
            a = hp.beta_a * a + (1.0 - hp.beta_a) * (g - gp)
            m, gp = hp.momentum * m + g + hp.alpha * a, g
        assert H.rel_max(ends[0][1][i].double().cpu().numpy(), m.numpy()) <= tol, (i, s)


def test_a_norm_out_of_range_in_a_small_step():
    """Tiny and not finite momenta beside an ordinary one: scaled, left alone, and untouched by the others."""
    print("[case] norms", flush=True)
    shapes = [(200, 300), (200, 301), (300, 200), (200, 300)]
    factors = [1e-25, 1e15, float("nan"), 1.0]
    weights = [wl.draw_weight(s, 300 + i, torch.float32, "cuda:0") for i, s in enumerate(shapes)]
    before = [w.clone() for w in weights]
    plain = [w.clone() for w in weights]
    opt, ref = B.MonaOptimizer(weights), B.MonaOptimizer(plain)
    grads = [wl.GradientStream(s, 400 + i, "cuda:0").next() for i, s in enumerate(shapes)]
    opt.step([g * f for g, f in zip(grads, factors)], wl.HParams())
    ref.step(grads, wl.HParams())
    assert opt.status() == [B.MONA_STATUS_RESCALED, B.MONA_STATUS_RESCALED, B.MONA_STATUS_NONFINITE, 0] and ref.status() == [0] * 4
    assert torch.equal(weights[2], before[2]) and torch.equal(weights[3], plain[3])
    for i in (0, 1):
        # the orthogonalised matrix does not depend on the scale; the roundings of the copies do, and each of the two is within the suite's
        # bound of the exact one
        moved, want = weights[i] - before[i], plain[i] - before[i]
        assert float((moved - want).norm() / want.norm()) <= 2 * H.TOL_NS_BF16, i
