"""Chains whose products have a buffer each and no flags (ns_chain_kernel): what the host lays out for them, followed without a GPU,
and on the GPU against the same chains with flags, which add up in the same order."""
import dataclasses
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


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [1, 4, 5])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shapes", [[(256, 512)], [(31, 33), (129, 97), (65, 300), (3, 1), (64, 32)], [(513, 520)], [(200, 1400), (161, 160)]])
def test_a_fresh_chain_gives_the_bits_of_one_with_flags(shapes, precision, steps):
    print(f"[case] {shapes} precision {precision} steps {steps}", flush=True)
    dev = "cuda:0"
    hp = dataclasses.replace(wl.HParams(), ns_steps=steps)
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
        ends.append(weights)
        del others
    for i, (x, y) in enumerate(zip(*ends)):
        assert torch.equal(x, y), i
