"""What the compiler makes of the memory-bound quantizer kernels, read from the
assembly of csrc/quantize.hip as the library is built: no GPU, and no timing."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_21849_amd import build as qbuild

pytestmark = pytest.mark.skipif(not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")),
                                reason="hipcc not available")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled kernel name -> its instructions."""
    out = str(tmp_path_factory.mktemp("isa") / "quantize.s")
    subprocess.run([qbuild.HIPCC, *qbuild.COMMON, "--cuda-device-only", "-S", os.path.join(qbuild.CSRC, "quantize.hip"),
                    "-o", out], check=True, capture_output=True)
    found, name = {}, None
    for line in open(out):
        m = re.match(r"(_ZN2qg\w+):", line)
        if m:
            name = m.group(1)
            found[name] = []
        elif name and line.startswith("\t") and not line.startswith("\t."):
            found[name].append(line.strip())
        elif line.startswith(".Lfunc_end"):
            name = None
    return found


def test_mx_rows_of_any_alignment_load_a_unit_at_once(kernels):
    # a thread's eight bf16 elements: one 16-byte load, not eight 2-byte ones
    mine = {n: k for n, k in kernels.items() if "10k_quant_mxI" in n}
    assert len(mine) == 2
    for name, code in mine.items():
        loads = [i.split()[0] for i in code if i.startswith("global_load")]
        assert loads == ["global_load_dwordx4"], (name, loads)


def test_dequantizers_store_adjacent_runs(kernels):
    # an aligned output: a lane writes 8 elements, so one 16-byte store of bf16, two adjacent ones of fp32 (more
    # elements a lane leave gaps between the lanes' pieces that no store of the same instruction fills)
    wide = {n: k for n, k in kernels.items() if re.search(r"k_dequant_(mxILb[01]ELb([01])E|(fp8|nvfp4)ILb([01])ELb1E)", n)}
    assert len(wide) == 8
    for name, code in wide.items():
        f32 = bool(re.search(r"k_dequant_(mxILb[01]ELb1E|(fp8|nvfp4)ILb1ELb1E)", name))
        stores = [i for i in code if i.startswith("global_store_dwordx4")]
        offsets = {int(m.group(1)) if (m := re.search(r"offset:(\d+)", i)) else 0 for i in stores}
        assert offsets == ({0, 16} if f32 else {0}), (name, stores)
        if "k_dequant_fp8" not in name:  # (FP8 tensors may end in single elements)
            assert len(stores) == len([i for i in code if i.startswith("global_store")]), name


def test_fp8_tensors_that_end_in_part_of_a_block(kernels):
    # codes without 16-byte alignment, or rows times columns no multiple of 16: whole 8-element units in 8-byte stores;
    # only the last 1 to 7 elements of a dense tensor one by one (a slice's rows are whole units)
    for h in (1, 2):
        code = {}
        for dense in (0, 1):
            (code[dense],) = [k for n, k in kernels.items() if "13k_quant_unitsILi1ELi%dELb%dELb0E" % (h, dense) in n]
            ops = [i.split()[0] for i in code[dense]]
            assert ops.count("global_store_dwordx2") == 2 * h, (h, dense)
            single = [sum(o.startswith(p) for o in ops) for p in ("global_load_ushort", "global_store_byte")]
            assert single == ([7 * h, 7 * h] if dense else [0, 0]), (h, dense, single)
