"""The persistent large-tile GEMMs at each height of their tiles (256, 192 and 128
rows, chosen by the number of rounds on 256 CUs), with odd and even chunk counts
and ragged last tiles: every output type through the epilogue test, and the fp32
values against the oracle at rows on both sides of every tile height's edges."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21849_amd as q
import synth
from gpu_util import check_linear, log, to_dev_bf16
from test_gpu_tile_epilogues import FMTS, test_ragged_tiles_every_output as every_output

pytestmark = pytest.mark.gpu

# on 256 CUs: 2420 x 5136 takes 256-row tiles (FP8 288 x 192, 256 rows at 1777 x
# 7008 instead), 1230 x 8208 192, 1900 x 4112 128
SHAPES = [(2420, 5136), (1230, 8208), (1900, 4112)]


@pytest.mark.parametrize("kind,k", [("nvfp4", 256), ("mxfp4", 512), ("mxfp8", 256), ("fp8", 1024), ("w4a16", 256)])
@pytest.mark.parametrize("m,n", SHAPES)
def test_every_output(kind, m, n, k):
    every_output(kind, m, n, k)


@pytest.mark.parametrize("kind,k", [("nvfp4", 128), ("nvfp4", 384), ("nvfp4", 640), ("mxfp4", 256), ("mxfp4", 768),
                                    ("mxfp4", 1024), ("mxfp8", 512), ("mxfp8", 768),
                                    ("fp8", 1024), ("fp8", 1152), ("w4a16", 384), ("w4a16", 512)])
@pytest.mark.parametrize("m,n", SHAPES + [(1777, 7008)])
def test_values_at_tile_edges(kind, m, n, k):
    log("tile heights %s m=%d n=%d k=%d" % (kind, m, n, k))
    x = synth.normal_bf16(m, k, 1.0, 52, 0)
    w = synth.normal_bf16(n, k, 0.02, 52, 1)
    fmt = FMTS[kind]
    a = to_dev_bf16(x) if kind == "w4a16" else q.quantize(to_dev_bf16(x), fmt)
    y = q.linear(a, q.pack(q.quantize(to_dev_bf16(w), fmt)), fmt, n, out_dtype=q.QG_OUT_F32)
    torch.cuda.synchronize()
    edges = sorted({e + d for h in (128, 192, 256) for e in range(0, m + 1, h) for d in (-1, 0, 31, 32)} | {m - 1})
    rows = np.array([e for e in edges if 0 <= e < m])
    cols = (np.arange(rows.size) * 797 + 255) % n
    check_linear(y, oracle.linear_reference(kind, x, w, rows, cols), rows, cols)
