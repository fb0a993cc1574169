"""Host check of apply_H's launch choice, without a GPU (tests/host/apply_plan_check.cpp):
after a product of one block width and pairing of its columns, a call that may
build no tables finds a route for any other width and pairing that a rule tied to
the tile alone would serve, within the scratch it has; and the columns per
workgroup and tile order asked for with automatic tiles reach every plan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_05725_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_launch_choice(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "apply_plan_check")
    # device code is only compiled to link; nothing of it runs
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-Xarch_device", "-O0", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "apply_plan_check.cpp"),
           os.path.join(CSRC, "terms.cpp"), os.path.join(CSRC, "timing.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
