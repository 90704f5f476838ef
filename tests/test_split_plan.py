"""Host-only check of which GEMM kernel a shape takes (plan_* in
csrc/tile_plan.hpp) against the measurements the rules rest on. No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_measured_shapes_take_their_tiling(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "split_plan_check")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++20",
                    "-I" + os.path.join(ROOT, "paper_2609_21849_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "split_plan_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "violations 0" in r.stdout, r.stdout[-2000:]
