"""The repair of a working copy (a norm out of range, or not finite) in the launch that begins a small step."""
import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(512, 1408), (300, 517), (96, 200)])
def test_chunks_that_share_lines_of_m(shape):
    """M is 16-byte aligned at least (mona_step_noalloc), so two chunks of it, 16 KB each, may meet within a 128-byte line, of which every die
    that had it keeps a copy: the repaired copies are those of an M whose chunks begin with a line, bit for bit."""
    dev = "cuda:0"
    hpc, stream = B.make_hparams(wl.HParams()), torch.cuda.current_stream().cuda_stream
    n = shape[0] * shape[1]
    grads = wl.GradientStream(shape, 41, dev)
    grads = [grads.next() * f for f in (1e-25, 3e-25, 1e-24, 1e16, 1e-23, 2e16)]
    w0 = wl.draw_weight(shape, 40, torch.float32, dev)
    ends = []
    for offset in (0, 16, 48, 64, 112):
        print(f"[case] {shape}, M {offset} bytes into a line", flush=True)
        room = torch.zeros(n + 64, dtype=torch.float32, device=dev)
        first = (-room.data_ptr() % 128 + offset) // 4
        mom = room[first:first + n]
        assert mom.data_ptr() % 128 == offset
        w, g_prev, acc = w0.clone(), torch.zeros(shape, device=dev), torch.zeros(shape, device=dev)
        for k, g in enumerate(grads):
            B.mona_step_noalloc(B.make_matrices([w], [g]), None, g_prev.data_ptr(), acc.data_ptr(), mom.data_ptr(), hpc, k, stream)
        torch.cuda.synchronize()
        ends.append((w, mom.clone()))
        assert torch.isfinite(w).all() and not torch.equal(w, w0)
        assert torch.equal(ends[0][0], w) and torch.equal(ends[0][1], ends[-1][1])


def spoil(g, how):
    """A gradient whose norm, or that of some of its chunks of 4096 elements, is out of range."""
    g = g.clone()
    flat = g.view(-1)
    if how == "all tiny":
        g.mul_(1e-25)
    elif how == "tiny, some chunks zero":
        g.mul_(1e-25)
        flat[: flat.numel() // 3].zero_()
    elif how == "some chunks tiny":              # (the norm is not)
        flat[flat.numel() // 2:].mul_(1e-25)
    elif how == "all large":
        g.mul_(1e16)
    elif how == "one large":
        flat[-2] = 1e20
    elif how == "one not a number":
        flat[flat.numel() // 2] = float("nan")
    elif how == "all zero":
        g.zero_()
    return g


HOW = ["all tiny", "tiny, some chunks zero", "some chunks tiny", "all large", "one large", "one not a number", "all zero", "ordinary"]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shapes", [[(512, 1408)], [(300, 517)], [(67, 61)], [(129, 260), (257, 257), (3, 5), (192, 136)]])
def test_shared_repair_gives_what_launches_of_their_own_give(shapes, precision):
    """The same bits as the pass, the norms and the repair in launches of their own (profiling level 2), for one norm after another on one
    state: the counters that the workgroups share are back at zero for each step."""
    dev = "cuda:0"
    hp = wl.HParams(flags=B.MONA_FLAG_KEEP_O)
    flagged = {"all tiny": B.MONA_STATUS_RESCALED, "tiny, some chunks zero": B.MONA_STATUS_RESCALED, "all large": B.MONA_STATUS_RESCALED,
               "one large": B.MONA_STATUS_RESCALED, "one not a number": B.MONA_STATUS_NONFINITE, "all zero": B.MONA_STATUS_ZERO_NORM}
    opts = []
    for level in (0, 2):
        opts.append(B.MonaOptimizer([wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)], ns_precision=precision))
        opts[-1].set_profiling(level)
    grads = [[wl.GradientStream(s, 400 + 50 * k + i, dev).next() for i, s in enumerate(shapes)] for k in range(2)]
    for turn in range(len(HOW)):
        # (each matrix of a list another norm)
        how = [HOW[(turn + 3 * i) % len(HOW)] for i in range(len(shapes))]
        print(f"[case] {shapes} precision {precision} {how}", flush=True)
        for opt in opts:
            for i in range(len(shapes)):
                for view in (opt.g_prev, opt.accel, opt.momentum):
                    view(i).zero_()
            for g in grads:
                opt.step([spoil(x, h) for x, h in zip(g, how)], hp)
        torch.cuda.synchronize()
        status = [flagged.get(h, 0) for h in how]
        for i, s in enumerate(shapes):
            if how[i] == "tiny, some chunks zero" and s[0] * s[1] < 100:
                continue
            assert opts[0].status()[i] == status[i], how[i]
        assert opts[0].status() == opts[1].status()
        for i in range(len(shapes)):
            same = [torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a, b.view(torch.int32) if b.dtype == torch.float32 else b)
                    for a, b in ((opts[0].weights[i], opts[1].weights[i]), (opts[0].momentum(i), opts[1].momentum(i)),
                                 (opts[0].last_o(i).contiguous(), opts[1].last_o(i).contiguous()))]
            assert all(same), (shapes[i], how[i], same)


@pytest.mark.parametrize("shape", [(512, 1408), (512, 2048), (513, 801)])
def test_a_small_step_with_a_repair_takes_little_longer(shape):
    """A repair reads M and writes the copy once more, 6 bytes an element, by all workgroups of the pass: a few us of a step of 90 to 105.  (By one
    workgroup alone it took 200 to 330.)  The bound leaves room for as much again as half the step."""
    dev = "cuda:0"
    hp = B.make_hparams(wl.HParams())
    w = [wl.draw_weight(shape, 300, torch.float32, dev)]
    base = [[wl.GradientStream(shape, 400 + k, dev).next()] for k in range(2)]
    times = {}
    for how in ("ordinary", "all tiny", "all large", "one large", "one not a number"):
        opt = B.MonaOptimizer(w)
        grads = [[spoil(g, how) for g in gs] for gs in base]
        best = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for k in range(40):
                opt.step(grads[k & 1], hp)
            b.record()
            b.synchronize()
            best.append(a.elapsed_time(b) * 1e3 / 40)
        times[how] = min(best[1:])
    print(f"[repair] {shape} us a step: {times}", flush=True)
    assert max(times.values()) < 1.5 * times["ordinary"], times
