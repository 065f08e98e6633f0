"""Chains whose products have a buffer each and no flags (ns_chain_kernel): what the host lays out for them, followed without a GPU,
and on the GPU against the same chains with flags, which add up in the same order."""
import ctypes
import dataclasses
import gc
import os
import subprocess

import pytest
import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl
from tests.test_host_launches import CLANG, HERE, OBJECTS


@pytest.mark.skipif(not all(map(os.path.exists, OBJECTS + [CLANG])), reason="library objects not built")
def test_buffers_of_a_fresh_chain(tmp_path):
    exe = str(tmp_path / "fresh_plan")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(HERE, "fresh_plan.cpp"),
                    os.path.join(HERE, "fake_hip.cpp"), *OBJECTS, "-o", exe], check=True, timeout=120)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr


def kind(opt):
    """Of the last step's chains: 1 with a buffer for every product, 0 with flags."""
    return opt.lib.mona_internal_chain_kind(ctypes.c_void_p(opt.state))


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [1, 4, 5])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shapes", [[(256, 512)], [(31, 33), (129, 97), (65, 300), (3, 1), (64, 32)], [(513, 520)], [(200, 1400), (161, 160)]])
def test_a_fresh_chain_gives_the_bits_of_one_with_flags(shapes, precision, steps):
    print(f"[case] {shapes} precision {precision} steps {steps}", flush=True)
    dev = "cuda:0"
    hp = dataclasses.replace(wl.HParams(), ns_steps=steps)
    gc.collect()                                 # (states that other tests have left)
    ends = []
    for full in (False, True):
        # (of 128 MB a state of 768 x 768 takes 16.5 and one of 256 x 256 two: no room is left for any of these)
        others = []
        while full and len(others) < 40:
            side = 768 if len(others) < 8 else 256
            others.append(B.MonaOptimizer([wl.draw_weight((side, side), 1, torch.float32, dev)]))
        weights = [wl.draw_weight(s, 300 + i, torch.float32, dev) for i, s in enumerate(shapes)]
        opt = B.MonaOptimizer(weights, ns_precision=precision)
        for k in range(3):
            grads = [wl.GradientStream(s, 400 + 50 * k + i, dev).next() for i, s in enumerate(shapes)]
            if k == 1:
                grads[0][0, 0] = -1e38           # the norm leaves the range of its square, the others' bits stay as they were
            opt.step(grads, hp)
        torch.cuda.synchronize()
        assert kind(opt) == (0 if full else 1)
        ends.append(weights)
        del others
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), i


@pytest.mark.gpu
def test_parts_given_back_while_steps_are_on_their_way():
    """States that are freed behind steps that have not run yet, and others that take their parts at once, on another stream."""
    print("[case] parts given back", flush=True)
    dev, shape, hp = "cuda:0", (768, 768), wl.HParams()
    gc.collect()
    grads = [wl.GradientStream(shape, 400 + i, dev).next() for i in range(6)]
    start = [wl.draw_weight(shape, 300 + i, torch.float32, dev) for i in range(6)]
    want = [w.clone() for w in start]
    for w, g in zip(want, grads):
        opt = B.MonaOptimizer([w])
        for _ in range(3):
            opt.step([g], hp)
        torch.cuda.synchronize()
        assert kind(opt) == 1
        del opt
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    kept, ends = [], [w.clone() for w in start]
    for turn in range(4):                        # (six of them to 128 MB, so the second turn needs what the first has given back)
        with torch.cuda.stream(streams[turn & 1]):
            opts = [B.MonaOptimizer([w]) for w in ends]
            for w, w0 in zip(ends, start):
                w.copy_(w0)
            for _ in range(3):
                for opt, g in zip(opts, grads):
                    opt.step([g], hp)
        assert [kind(opt) for opt in opts] == [1] * 6
        kept += [(opt.arena, ends) for opt in opts]
        for opt in opts:
            opt.close()
        results = ends
        ends = [w.clone() for w in start]
        kept.append(results)
    torch.cuda.synchronize()
    for results in kept:
        if isinstance(results, list):
            for i, (x, y) in enumerate(zip(results, want)):
                assert torch.equal(x, y), i


@pytest.mark.gpu
def test_a_graph_replayed_after_its_state_is_freed():
    """The recorded step needs the arena and the arrays it names; a state made afterwards gets other buffers, and both may run side by side."""
    print("[case] replay after free", flush=True)
    dev, shape, hp = "cuda:0", (256, 512), wl.HParams()
    gc.collect()
    grad = wl.GradientStream(shape, 400, dev).next()
    ends = []
    for use_graph in (False, True):
        w, other = (wl.draw_weight(shape, 300 + i, torch.float32, dev) for i in range(2))
        opt = B.MonaOptimizer([w])
        opt.step([grad], hp)
        torch.cuda.synchronize()
        if use_graph:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                opt.step([grad], hp)
            arena = opt.arena
            opt.close()
        second = B.MonaOptimizer([other])
        assert not use_graph or arena.data_ptr() != second.arena.data_ptr()
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        for _ in range(20):
            if use_graph:
                graph.replay()
            else:
                opt.step([grad], hp)
            with torch.cuda.stream(side):
                second.step([grad], hp)
        torch.cuda.synchronize()
        assert second.status() == [0]
        ends.append((w, other))
    for x, y in zip(*ends):
        assert torch.equal(x, y)
