"""Host-only check of the unit-to-row multiplication that the quantizers use for
column slices (csrc/quant_plan.hpp) against the division. No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_row_of_unit_equals_division(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "unit_rows_check")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++20",
                    "-I" + os.path.join(ROOT, "paper_2609_21849_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "unit_rows_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "violations 0" in r.stdout, r.stdout[-2000:]
    assert int(r.stdout.split("checked ")[1].split()[0]) > 50000
