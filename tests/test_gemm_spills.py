"""Registers that the GEMM kernels keep in scratch memory, from the metadata of
the built library: a reload at the start of a tile waits for the stores of the
tile before it. No GPU."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2609_21849_amd as q

LLVM = "/opt/rocm/llvm/bin"


def _code_objects(blob):
    """The gfx950 code objects of a library's .hip_fatbin section (one bundle per source)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        p = at + len(magic)
        (count,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name:
                yield blob[at + offset:at + offset + size]
        at = blob.find(magic, at + 1)


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """Mangled kernel name -> spilled vector registers."""
    if not os.path.exists(q.LIB_PATH):
        pytest.skip("libqgemm.so is not built")
    tools = [shutil.which(t) or os.path.join(LLVM, t) for t in ("llvm-objcopy", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("llvm tools not available")
    d = tmp_path_factory.mktemp("co")
    subprocess.run([tools[0], "--dump-section", ".hip_fatbin=%s" % (d / "fat"), q.LIB_PATH, os.devnull], check=True)
    found = {}
    for i, co in enumerate(_code_objects((d / "fat").read_bytes())):
        (d / ("co%d" % i)).write_bytes(co)
        notes = subprocess.run([tools[1], "--notes", str(d / ("co%d" % i))], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"^ {4}\.name:\s+(\S+)$", notes, re.M)
        counts = re.findall(r"\.vgpr_spill_count:\s+(\d+)", notes)
        assert len(names) == len(counts)
        found.update(zip(names, map(int, counts)))
    return found


def test_large_tiles_keep_their_registers(spills):
    # template arguments: epilogue (0 to 3 staged in LDS, 4 element by element), tile height / 64
    tiles = {n: s for n, s in spills.items() if re.search(r"k_gemm_\w+_directILi[0-3]ELi[234]E", n)}
    assert len(tiles) == 5 * 3 * 4 - 3  # (no NVFP4 output for bf16 activations)
    over = {n: s for n, s in tiles.items() if s > (5 if "mxfp8_directILi3E" in n else 1)}
    assert not over, over


def test_other_gemm_kernels_spill_nothing(spills):
    rest = {n: s for n, s in spills.items() if re.search(r"k_gemm_(splitk|fp8)I|k_w4a16_|k_gemm_fp8_t288", n)}
    assert len(rest) > 20 and not any(rest.values()), {n: s for n, s in rest.items() if s}
