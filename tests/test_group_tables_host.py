"""Host check of the 16-row apply kernel's tables, without a GPU:
tests/host/group_tables_emu.cpp builds them with the library's host code and
evaluates H psi from them the way the kernel reads them (full space and both
parity sectors, one and two row layouts, both element sizes), against the
direct sum over the term tables; up to N = 60 the builder alone runs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_05725_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_group_tables_match_direct_sum(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "group_tables_emu")
    # device code is only compiled to link; nothing of it runs
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-Xarch_device", "-O0", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "group_tables_emu.cpp"),
           os.path.join(CSRC, "terms.cpp"), os.path.join(CSRC, "timing.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
    assert sum("rel_err" in ln for ln in r.stdout.splitlines()) > 30
