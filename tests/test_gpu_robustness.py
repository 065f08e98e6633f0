"""GPU tests of the cases a long training run meets sooner or later: gradients of extreme scale, a matrix
that stops receiving gradients, a NaN step followed by a restored checkpoint, memory next to the arena."""
import ctypes as C
import dataclasses

import numpy as np
import pytest
import torch

from oracle import mona_oracle as orc
from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.mark.parametrize("scale", [1e-25, 1e-14, 1e-9, 1e15, 1e30])
def test_gradient_scale_does_not_matter(scale):
    """X_0 = M / ||M||_F (Sec. 3.2) is scale-free: gradients of any magnitude the fp32 state can hold must give
    the oracle's O.  (The products accumulate the unscaled working copy in fp32; outside the safe window of
    the norm the copy is rescaled by a power of two first.)"""
    say(f"[case] gradient scale {scale:g}")
    shapes = [(256, 512), (300, 100), (40, 64), (512, 1536)]
    weights = [wl.draw_weight(s, 5000 + i, torch.float32) for i, s in enumerate(shapes)]
    streams = [wl.GradientStream(s, 5100 + i, sigma=scale) for i, s in enumerate(shapes)]
    grads = [[st.next() for st in streams] for _ in range(2)]
    hp = wl.HParams()
    opt, _, hist = H.run_gpu(weights, grads, hp, 0)
    worst = H.check_history(weights, grads, hp, hist, range(len(shapes)), H.TOL_NS_BF16, label=f"scale {scale:g}")
    say("[worst]", worst)
    st = opt.status()
    for i, s in enumerate(st):
        norm = float(np.sqrt((hist[-1][i].M ** 2).sum()))
        assert ((s & B.MONA_STATUS_RESCALED) != 0) == (not 2.0 ** -40 <= norm <= 2.0 ** 40), (i, s, norm)
        assert (s & 3) == 0
    assert any(s & B.MONA_STATUS_RESCALED for s in st) == (scale != 1e-9)


def test_matrix_without_gradients_decays_to_zero_cleanly():
    """A matrix that receives exactly zero gradients (a dead expert): M decays as mu^k, G~ = alpha A decays
    as beta_a^k.  O must follow the oracle all the way down, through the rescaled range, until M is exactly
    zero, where only weight decay is left."""
    say("[case] zero gradients from step 2 on")
    shape = (192, 320)
    dev = "cuda:0"
    w = wl.draw_weight(shape, 5200, torch.float32, dev)
    g1 = wl.GradientStream(shape, 5201, dev).next()
    zero = torch.zeros(shape, device=dev)
    hp = wl.HParams(momentum=0.5, beta_a=0.5, alpha=-1.0, flags=B.MONA_FLAG_KEEP_O)
    ohp = H.oracle_hp(hp)
    opt = B.MonaOptimizer([w])
    o = orc.MonaOracle(shape)
    seen_rescaled = seen_zero = False
    for k in range(200):
        g = g1 if k == 0 else zero
        opt.step([g], hp)
        M = o.elementwise(H.f64(g), ohp)
        st = opt.status()[0]
        m_gpu = H.f64(opt.momentum(0))
        if not m_gpu.any():
            seen_zero = True
            assert st == B.MONA_STATUS_ZERO_NORM
            assert not H.f64(opt.last_o(0)).any()
            break
        if k % 8 == 0 or (st & B.MONA_STATUS_RESCALED):
            # fp32 state: compare O against the oracle's Newton-Schulz of the GPU's own M (the state arrays
            # leave the oracle's float64 trajectory once they reach fp32 subnormals)
            O_ref = orc.newton_schulz(m_gpu, ohp.ns_steps, ohp.ns_a, ohp.ns_b, ohp.ns_c, ohp.ns_eps)
            e = H.rel_fro(H.f64(opt.last_o(0)), O_ref)
            nrm = float(np.sqrt((m_gpu ** 2).sum()))
            assert e <= H.TOL_NS_BF16, f"step {k + 1}: ||M|| = {nrm:.3e}, O rel Fro err {e:.3e}"
            assert abs(float(opt.norm(0).item()) - nrm) <= 1e-6 * nrm + 2.0 ** -149    # the norm is reported in fp32
            if st & B.MONA_STATUS_RESCALED:
                seen_rescaled = True
                assert nrm < 2.0 ** -40
    assert seen_rescaled and seen_zero
    assert torch.isfinite(w).all()


def test_nan_step_then_restored_checkpoint_on_a_ragged_shape():
    """A NaN gradient must not outlive the step it came in: the parameter is left alone, and once the caller
    restores the previous checkpoint the following clean step is the oracle's (no NaN may have reached the
    zero padding of the working matrices, which a 333 x 130 matrix has on every side)."""
    say("[case] NaN step, import, clean step")
    shapes = [(333, 130), (100, 300), (512, 1536)]
    dev = "cuda:0"
    weights = [wl.draw_weight(s, 5300 + i, torch.float32) for i, s in enumerate(shapes)]
    streams = [wl.GradientStream(s, 5310 + i) for i, s in enumerate(shapes)]
    grads = [[st.next() for st in streams] for _ in range(3)]
    hp = wl.HParams()
    dev_w = [w.to(dev) for w in weights]
    opt = B.MonaOptimizer(dev_w)
    hpk = dataclasses.replace(hp, flags=B.MONA_FLAG_KEEP_O)
    opt.step([g.to(dev) for g in grads[0]], hpk)
    ckpt = opt.export_state().clone()
    w_before = [w.clone() for w in dev_w]
    bad = [g.clone() for g in grads[1]]
    for b in bad:
        b[7, 9] = float("nan")
    opt.step([g.to(dev) for g in bad], hpk)
    assert all(s & B.MONA_STATUS_NONFINITE for s in opt.status())
    for w0, w1 in zip(w_before, dev_w):
        assert torch.equal(w0, w1)
    opt.import_state(ckpt, 1)
    opt.step([g.to(dev) for g in grads[1]], hpk)
    torch.cuda.synchronize()
    assert opt.status() == [0, 0, 0]
    ref = H.run_oracle_for(weights, grads[:2], hp, range(3))
    for i in range(3):
        assert H.rel_max(H.f64(opt.momentum(i)), ref[i][1]["M"]) <= H.TOL_STATE
        e = H.rel_fro(H.f64(opt.last_o(i)), ref[i][1]["O"])
        assert e <= H.TOL_NS_BF16, (i, e)
        assert torch.isfinite(dev_w[i]).all()
    # also without the import: the NaN momentum stays flagged, and a repaired M gives a clean step
    opt2 = B.MonaOptimizer([w.to(dev) for w in weights])
    opt2.step([g.to(dev) for g in bad], hpk)
    for i in range(3):
        opt2.momentum(i).zero_(); opt2.accel(i).zero_(); opt2.g_prev(i).zero_()
    opt2.step([g.to(dev) for g in grads[0]], hpk)
    torch.cuda.synchronize()
    assert opt2.status() == [0, 0, 0]
    for i in range(3):
        e = H.rel_fro(H.f64(opt2.last_o(i)), ref[i][0]["O"])
        assert e <= H.TOL_NS_BF16, (i, e)


def test_nothing_is_written_outside_the_arena():
    """Canary words on both sides of the arena survive init, steps of every kernel kind and a checkpoint
    round trip."""
    say("[case] arena canaries")
    dev = "cuda:0"
    shapes = [(512, 1536)] * 12 + [(333, 130), (100, 300), (40, 64), (257, 257)]
    weights = [wl.draw_weight(s, 5400 + i, torch.bfloat16, dev) for i, s in enumerate(shapes)]
    grads = [wl.GradientStream(s, 5410 + i, dev).next() for i, s in enumerate(shapes)]
    mats = B.make_matrices(weights, None)
    need = B.mona_state_size(mats, len(shapes))
    guard = 1 << 20
    buf = torch.full((need + 2 * guard,), 0xA5, dtype=torch.uint8, device=dev)
    arena = buf[guard: guard + need]
    assert arena.data_ptr() % 256 == 0
    s = torch.cuda.current_stream().cuda_stream
    state = B.mona_init_state(mats, len(shapes), None, arena, s)
    for T in (5, 0):
        hp = B.make_hparams(wl.HParams(ns_steps=T, flags=B.MONA_FLAG_KEEP_O))
        B.mona_step(state, B.make_matrices(weights, grads), len(shapes), hp, s)
    torch.cuda.synchronize()
    B.mona_free_state(state)
    assert bool((buf[:guard] == 0xA5).all()) and bool((buf[guard + need:] == 0xA5).all())


def test_alpha_outside_the_theorems_range_is_noted_not_refused():
    say("[case] alpha warning")
    dev = "cuda:0"
    w = [wl.draw_weight((64, 96), 5500, torch.float32, dev)]
    g = [wl.GradientStream((64, 96), 5501, dev).next()]
    opt = B.MonaOptimizer(w)
    lib = B.load_library()
    opt.step(g, wl.HParams(beta_a=0.9, alpha=-5.0))
    assert lib.mona_last_error() == b""
    opt.step(g, wl.HParams(beta_a=0.9, alpha=-10.0))          # |alpha| = 1 / (1 - beta_a): not below it
    msg = lib.mona_last_error().decode()
    assert msg.startswith("warning") and "1 / (1 - beta_a)" in msg
    assert opt.step_count() == 2
    opt.step(g, wl.HParams(beta_a=0.9, alpha=-10.0, flags=B.MONA_FLAG_MUON_ONLY))   # alpha is ignored there
    assert lib.mona_last_error() == b""
    torch.cuda.synchronize()


@pytest.mark.parametrize("rest, shape", [(0, (257, 1001)), (600, (257, 1001)), (600, (1024, 700)), (64, (300, 1000)),
                                         (2100, (130, 70))])
@pytest.mark.parametrize("precision", [0, 1])
def test_repair_of_one_flagged_matrix_in_a_list(rest, shape, precision):
    """The working copy of a matrix whose norm is out of range is rewritten in the launch that forms the norms, or in a
    launch of its own where the list is too long for that: either way O is the oracle's, a non-finite matrix
    leaves everything else alone, and the zero padding survives."""
    say(f"[case] {rest} small matrices and one {shape}, precision {precision}")
    dev = "cuda:0"
    shapes = [(12 + i % 5, 20 + i % 7) for i in range(rest)] + [shape]
    weights = [wl.draw_weight(s, 5600 + i, torch.float32) for i, s in enumerate(shapes)]
    grads = [wl.GradientStream(s, 5700 + i).next() for i, s in enumerate(shapes)]
    watch = [len(shapes) - 1] + ([0] if rest else [])
    tol = H.TOL_NS_F32 if precision else H.TOL_NS_BF16
    hp = dataclasses.replace(wl.HParams(), flags=B.MONA_FLAG_KEEP_O)
    dev_w = [w.to(dev) for w in weights]
    opt = B.MonaOptimizer(dev_w, ns_precision=precision)
    start = opt.export_state().clone()

    def step(last):
        gs = grads[:-1] + [last]
        opt.step([g.to(dev) for g in gs], hp)
        torch.cuda.synchronize()
        return gs

    for scale in (1e-25, 1e18):
        gs = step(grads[-1] * scale)
        assert opt.status() == [0] * rest + [B.MONA_STATUS_RESCALED]
        ref = H.run_oracle_for(weights, [gs], hp, watch)
        for i in watch:
            assert H.rel_fro(H.f64(opt.last_o(i)), ref[i][0]["O"]) <= tol, (scale, i)
        opt.import_state(start, 0)
    before = dev_w[-1].clone()
    bad = grads[-1].clone()
    bad[-1, -1] = float("nan")
    step(bad)
    assert opt.status() == [0] * rest + [B.MONA_STATUS_NONFINITE]
    assert torch.equal(before, dev_w[-1]) and not H.f64(opt.last_o(len(shapes) - 1)).any()
    # (no import here: it would clear the padding, which the repair must have left zero by itself)
    for view in (opt.g_prev, opt.accel, opt.momentum):
        view(len(shapes) - 1).zero_()
    step(grads[-1])
    ref = H.run_oracle_for(weights, [grads], hp, watch[:1])
    assert H.rel_fro(H.f64(opt.last_o(watch[0])), ref[watch[0]][0]["O"]) <= tol


@pytest.mark.parametrize("rest, shape", [(0, (4096, 1536)), (64, (4096, 1536)), (600, (4096, 1536))])
def test_repair_does_not_hold_up_the_step(rest, shape):
    """A flagged matrix costs one more pass over it, by the whole chip, whatever the length of the list: 25 MB read and
    13 written, 10 us at 4 TB/s.  Half a millisecond leaves room for one launch and for a quiet chip; a repair
    whose width shrinks with the list took 12 ms."""
    say(f"[case] repair time, {rest} small matrices and one {shape}")
    dev = "cuda:0"
    shapes = [(16, 24)] * rest + [shape]
    weights = [torch.zeros(s, device=dev) for s in shapes]
    best = []
    for scale in (1.0, 1e-20):
        grads = [wl.GradientStream(s, 5800 + i, dev).next() for i, s in enumerate(shapes)]
        grads[-1].mul_(scale)
        opt = B.MonaOptimizer(weights)
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            opt.step(grads, wl.HParams())
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        assert opt.status() == [0] * rest + [0 if scale == 1.0 else B.MONA_STATUS_RESCALED]
        best.append(min(times[1:]))
    say(f"[repair] step {best[0]:.3f} ms, with one flagged matrix {best[1]:.3f} ms")
    assert best[1] - best[0] < 0.5


@pytest.mark.parametrize("shapes", [[(256, 512), (100, 300)], [(40, 72)] * 97])
def test_eager_steps_with_other_buffers_between_graph_replays(shapes):
    """A graph holds the pointers of the step that was recorded, and eager steps before, between and after its replays
    their own, with a table of at most and of more than 96 matrices."""
    say(f"[case] {len(shapes)} matrices, replays and eager steps with other buffers in turn")
    dev = "cuda:0"
    hp = wl.HParams()
    ends = []
    for use_graph in (False, True):
        weights = [wl.draw_weight(s, 5900 + i, torch.float32, dev) for i, s in enumerate(shapes)]
        buffers = [[wl.GradientStream(s, 6000 + 100 * k + i, dev).next() for i, s in enumerate(shapes)] for k in range(2)]
        opt = B.MonaOptimizer(weights)
        graph = None
        opt.step(buffers[0], hp)
        torch.cuda.synchronize()
        if use_graph:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                opt.step(buffers[0], hp)
            torch.cuda.synchronize()
        for k in range(3):
            opt.step(buffers[1], hp)
            opt.step(buffers[1], hp)
            if use_graph:
                graph.replay()
            else:
                opt.step(buffers[0], hp)
        opt.step(buffers[1], hp)
        torch.cuda.synchronize()
        ends.append(weights + [opt.momentum(i).clone() for i in range(len(shapes))])
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), i
