"""Which form of the elementwise pass and of the update of large tiles a step takes, by size, type and alignment (tests/host/kernel_forms.cpp)."""
import os
import subprocess

import pytest

from tests.test_host_launches import CLANG, HERE, OBJECTS


@pytest.mark.skipif(not all(map(os.path.exists, OBJECTS + [CLANG])), reason="library objects not built")
def test_forms_follow_size_type_and_alignment(tmp_path):
    exe = str(tmp_path / "kernel_forms")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(HERE, "kernel_forms.cpp"),
                    os.path.join(HERE, "fake_hip.cpp"), *OBJECTS, "-o", exe], check=True, timeout=120)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
