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
