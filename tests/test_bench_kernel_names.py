"""bench.py finds kernels in profiler output by name: every name it looks for is
a __global__ of the library, and --quant-summary reads a capture that holds the
library's own kernel names. No GPU."""
import csv
import glob
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernels():
    names = set()
    for f in glob.glob(os.path.join(ROOT, "paper_2609_21849_amd", "csrc", "*.hip")):
        names |= set(re.findall(r"__global__\s+void\s+(?:__launch_bounds__\([^)]*\)\s*)?(\w+)\s*\(", open(f).read()))
    return names


def test_every_name_is_a_kernel():
    kernels = _kernels()
    assert len(kernels) > 20
    missing = (set(bench.KERNEL.values()) | set(bench.QUANT_KERNELS)) - kernels
    assert not missing, missing


def _write(path, header, rows):
    os.makedirs(os.path.dirname(path))
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(header)
        w.writerows(rows)


def test_quant_summary_reads_the_librarys_kernels(tmp_path):
    # the chain of every call: amax, finalize, elements, in the order it launches
    src = open(os.path.join(ROOT, "paper_2609_21849_amd", "csrc", "quantize.hip")).read()
    chain = ["void qg::k_amax_units<true>(unsigned short const*)", "qg::k_finalize(unsigned int const*)",
             "void qg::k_quant_units<%d, 2, true, true>(unsigned short const*)"]
    for name in chain:
        assert "__global__" in src and re.search(r"\b%s\b" % re.search(r"k_\w+", name).group(), src)
    calls = [name % fmt if "%d" in name else name for fmt in (1, 2) for _ in bench.QUANT_SHAPES for _ in range(4)
             for name in chain]
    copy = ["__amd_rocclr_copyBuffer"] * 3
    kib = bench.COPY_BYTES // 1024
    for ctr in ("FETCH_SIZE", "WRITE_SIZE"):
        _write(str(tmp_path / ctr / "run_counter_collection.csv"), ["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"],
               [[i, n, ctr, kib if n in copy else 1000] for i, n in enumerate(calls + copy)])
    _write(str(tmp_path / "trace" / "run_kernel_trace.csv"), ["Kernel_Name", "Start_Timestamp", "End_Timestamp"],
           [[n, 100000 * i, 100000 * i + 5000] for i, n in enumerate(calls + copy)])
    out = tmp_path / "summary.md"
    bench.quant_summary(str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), str(tmp_path / "trace"), str(out))
    text = out.read_text()
    for name in bench.QUANT_KERNELS:
        assert text.count("| `%s` | 1.0 | 1.0 |" % name) == 2 * len(bench.QUANT_SHAPES)
