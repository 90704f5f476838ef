"""Every split-K tiling the dispatch picks for NVFP4, W4A16 and long-K FP8 on a
256-CU device, at ragged sizes on either side of each change of tiling, fp32
outputs against the CPU oracle (sampled at tile edges)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21849_amd as q
import synth
from gpu_util import check_linear, log, to_dev_bf16

pytestmark = pytest.mark.gpu

FP8, NVFP4, BF16 = q.QG_FMT_FP8_E4M3, q.QG_FMT_NVFP4, q.QG_FMT_BF16
KINDS = {"fp8": (FP8, FP8), "nvfp4": (NVFP4, NVFP4), "w4a16": (BF16, NVFP4)}
CASES = [("nvfp4", 33, 48, 384), ("nvfp4", 33, 48, 4224),               # 32 x 32, short and long K
         ("nvfp4", 300, 1008, 384), ("nvfp4", 40, 4112, 4224),          # 32 x 64, short and long K
         ("nvfp4", 256, 3056, 128),                                     # 32 x 96
         ("nvfp4", 500, 3072, 256),                                     # 64 x 96
         ("nvfp4", 1001, 3008, 128),                                    # 64 x 64, two a CU
         ("nvfp4", 593, 1392, 512),                                     # 64 x 64, eight waves, one a CU
         ("nvfp4", 1273, 1968, 5248),                                   # 64 x 96, several rounds
         ("w4a16", 1, 48, 3072), ("w4a16", 31, 8240, 3200),             # few rows
         ("w4a16", 40, 48, 3200),                                       # 32 x 32
         ("w4a16", 250, 3056, 1024),                                    # 32 x 64, four waves
         ("w4a16", 300, 1008, 1152),                                    # 32 x 64, eight waves
         ("w4a16", 200, 9200, 1152),                                    # 32 x 64 for the row padding
         ("w4a16", 500, 3072, 1152),                                    # 64 x 96
         ("w4a16", 1100, 2000, 256), ("w4a16", 2050, 336, 1152),        # 64 x 64
         ("w4a16", 2050, 336, 256),                                     # 32 x 64, four waves, many rows
         ("w4a16", 150, 21568, 3072),                                   # 64 x 64 for the large tiles' padding
         ("fp8", 500, 3072, 2048), ("fp8", 449, 3008, 2176)]            # 64 x 96


@pytest.mark.parametrize("kind,m,n,k", CASES)
def test_splitk_tiling_parity(kind, m, n, k):
    log("split-K tiling %s m=%d n=%d k=%d" % (kind, m, n, k))
    x = synth.normal_bf16(m, k, 1.0, 61, 0, outlier_frac=0.004, outlier_gain=30.0)
    w = synth.normal_bf16(n, k, 0.02, 61, 1)
    a_fmt, w_fmt = KINDS[kind]
    packed = q.pack(q.quantize(to_dev_bf16(w), w_fmt))
    a = to_dev_bf16(x) if a_fmt == BF16 else q.quantize(to_dev_bf16(x), a_fmt)
    buf = torch.full((m + 1, n), 77.0, device="cuda")
    y = q.linear(a, packed, w_fmt, n, out_dtype=q.QG_OUT_F32, y=buf[:m])
    torch.cuda.synchronize()
    assert bool((buf[m] == 77).all())
    rng = np.random.default_rng(m + n)
    er = np.array(sorted({min(v, m - 1) for b in range(0, m + 64, 64) for v in (b - 1, b, b + 31, b + 32) if v >= 0}))
    ec = np.array(sorted({min(v, n - 1) for t in (64, 96) for b in range(0, n + t, t) for v in (b - 1, b) if v >= 0}))
    rows = np.concatenate([rng.integers(0, m, ec.size), er, rng.integers(0, m, 600)])
    cols = np.concatenate([ec, rng.integers(0, n, er.size), rng.integers(0, n, 600)])
    check_linear(y, oracle.linear_reference(kind, x, w, rows, cols), rows, cols)
