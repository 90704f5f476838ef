"""The MX GEMM's split-K tilings (few tokens) against the CPU oracle: each
tiling that the dispatch picks on a 256-CU device, the sizes on either side of
the change to large tiles, ragged rows and columns, odd and even chunk
counts per wave, and the quantized outputs of its reduction epilogue."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21849_amd as q
import synth
from gpu_util import check_linear, host, log, to_dev_bf16

pytestmark = pytest.mark.gpu

MXFP4, MXFP8 = q.QG_FMT_MXFP4, q.QG_FMT_MXFP8
NAME = {MXFP4: "mxfp4", MXFP8: "mxfp8"}
SHAPES = [(1, 16, 256), (33, 48, 512),          # 32 x 32 tiles
          (300, 1008, 768),                     # 32 x 64
          (256, 3056, 256),                     # 32 x 96
          (500, 3072, 1280),                    # 64 x 96, one round
          (777, 2000, 512),                     # 64 x 128
          (1001, 3008, 256),                    # large tiles, 128 x 256
          (1089, 3072, 256),                    # large tiles, 128 x 256
          (700, 3008, 6400)]                    # MXFP8: 64 x 96, two rounds; MXFP4: large tiles


def _operands(m, n, k, fmt, seed):
    x = synth.normal_bf16(m, k, 1.0, seed, 0, outlier_frac=0.004, outlier_gain=30.0)
    w = synth.normal_bf16(n, k, 0.02, seed, 1)
    return x, w, q.quantize(to_dev_bf16(x), fmt), q.pack(q.quantize(to_dev_bf16(w), fmt))


@pytest.mark.parametrize("fmt", [MXFP4, MXFP8])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_mx_few_tokens_parity(fmt, m, n, k):
    log("%s few tokens m=%d n=%d k=%d" % (NAME[fmt], m, n, k))
    x, w, a, packed = _operands(m, n, k, fmt, 41)
    y = q.linear(a, packed, fmt, n, out_dtype=q.QG_OUT_F32)
    yb = q.linear(a, packed, fmt, n)
    torch.cuda.synchronize()
    check_linear(y, oracle.linear_reference(NAME[fmt], x, w))
    assert torch.equal(yb, y.bfloat16())        # the bf16 output is the rounding of the same sums


@pytest.mark.parametrize("fmt", [MXFP4, MXFP8])
@pytest.mark.parametrize("m,n,k", [(40, 48, 256), (500, 3072, 256)])
def test_mx_few_tokens_quantized_outputs(fmt, m, n, k):
    _, _, a, packed = _operands(m, n, k, fmt, 42)
    y = q.linear(a, packed, fmt, n, out_dtype=q.QG_OUT_F32)
    s8 = (y.abs().max() / 448.0).reshape(1)
    s4 = (y.abs().max() / 2688.0).reshape(1)
    q8 = q.linear_fp8_out(a, packed, fmt, n, s8)
    q4 = q.linear_nvfp4_out(a, packed, fmt, n, s4)
    torch.cuda.synchronize()
    want = (y * (1.0 / s8)).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    assert torch.equal(q8.codes, want)
    codes, scales = oracle.quantize_nvfp4_static_f32(host(y), float(host(s4)[0]))
    assert np.array_equal(host(q4.codes), codes) and np.array_equal(host(q4.block_scales), scales)
