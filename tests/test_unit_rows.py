"""Host-only checks of the quantizers' addressing (csrc/quant_plan.hpp): the
unit-to-row multiplication of column slices against the division, and the
pieces that very large tensors are launched in. No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, name):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++20",
                    "-I" + os.path.join(ROOT, "paper_2609_21849_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "violations 0" in r.stdout, r.stdout[-2000:]
    return int(r.stdout.split("checked ")[1].split()[0])


def test_row_of_unit_equals_division(tmp_path):
    assert _run(tmp_path, "unit_rows_check") > 50000


def test_pieces_of_large_tensors(tmp_path):
    assert _run(tmp_path, "pieces_check") > 100
