"""The launch that begins a small step: what the workgroup that finishes a matrix last reads of the others must not come from caches that no
kernel boundary has renewed.  Seen in the device code, because whether a stale line is met is a matter of chance."""
import os
import re
import subprocess

import pytest

from paper_2605_26842_amd import build


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_loads_behind_the_count_are_at_device_scope(tmp_path):
    out = str(tmp_path / "state_update.s")
    subprocess.run([build.hipcc_path(), f"--offload-arch={build.ARCH}", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "--cuda-device-only", "-S", os.path.join(build.CSRC, "state_update.hip"), "-o", out],
                   check=True, capture_output=True, timeout=300)
    with open(out) as f:
        text = f.read()
    bodies = re.findall(r"\n_ZN\S*begin_norm_finalize_kernel\S*:(.*?)\.Lfunc_end", text, re.S)
    assert len(bodies) == 5
    for body in bodies:
        counted = re.search(r"global_atomic_add v\d+.* sc0", body)          # the count of workgroups that have arrived
        behind = [line.strip() for line in body[counted.end():].splitlines() if re.match(r"\s*(global|buffer|flat)_load", line)]
        assert len(behind) > 2 and all(" sc1" in line for line in behind), behind
