"""What libmona's host code enqueues, followed without a GPU: its objects are linked with a stand-in for the HIP runtime
(tests/host/fake_hip.cpp) that works on host memory."""
import os
import subprocess

import pytest

from paper_2605_26842_amd import build

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")
OBJECTS = [os.path.join(build.HERE, "_build", s.replace(".hip", ".o")) for s in build.SOURCES]
CLANG = "/opt/rocm/lib/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not all(map(os.path.exists, OBJECTS + [CLANG])), reason="library objects not built")


@pytest.mark.parametrize("program", ["pointer_tables", "launch_plan", "chain_plan", "executed_flops", "matrix_plan",
                                     "device_queries", "kept_plan"])
def test_what_the_host_enqueues(program, tmp_path):
    exe = str(tmp_path / program)
    subprocess.run([CLANG, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, program + ".cpp"), os.path.join(HERE, "fake_hip.cpp"), *OBJECTS, "-o", exe],
                   check=True, timeout=120)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_host_code_under_sanitizers(tmp_path):
    out = subprocess.run(["bash", os.path.join(HERE, "run_sanitizers.sh"), str(tmp_path)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-3000:] + out.stderr[-3000:]
