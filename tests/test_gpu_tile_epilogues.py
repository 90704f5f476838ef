"""The staged epilogues of the large-tile GEMM kernels (bf16, fp32, FP8 codes,
NVFP4 codes and block scales) on outputs whose last tiles are ragged in both
directions, against the element-wise epilogue that unaligned outputs take: the
same accumulators, so the same bits; nothing written outside the output; the
fp32 values themselves against the oracle at tile edges."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21849_amd as q
import synth
from gpu_util import DEV, check_linear, host, log, to_dev_bf16

pytestmark = pytest.mark.gpu

FMTS = {"fp8": q.QG_FMT_FP8_E4M3, "nvfp4": q.QG_FMT_NVFP4, "mxfp4": q.QG_FMT_MXFP4, "mxfp8": q.QG_FMT_MXFP8,
        "w4a16": q.QG_FMT_NVFP4}
# on 256 CUs 1900 x 4112 takes tiles of 128 x 256, ragged in both directions: the
# last row tile holds 108 rows, the last column tile 16 (the taller tiles: see
# test_gpu_tile_heights.py); the second fp8 shape fills whole 256 x 256 tiles
CASES = [("fp8", 1900, 4112, 256), ("fp8", 2048, 8192, 128), ("nvfp4", 1900, 4112, 128), ("nvfp4", 1900, 4112, 256),
         ("mxfp4", 1900, 4112, 256), ("mxfp8", 1900, 4112, 256), ("w4a16", 1900, 4112, 256)]


def _gemm_args(a, packed, fmt, n, k):
    if isinstance(a, q.QTensor):
        return (a.fmt, a.codes, a.block_scales, a.tensor_scale, k, fmt, packed, packed.numel(), a.rows, n, k)
    return (q.QG_FMT_BF16, a, None, None, k, fmt, packed, packed.numel(), a.shape[0], n, k)


@pytest.mark.parametrize("kind,m,n,k", CASES)
def test_ragged_tiles_every_output(kind, m, n, k):
    log("tile epilogues %s m=%d n=%d k=%d" % (kind, m, n, k))
    fmt = FMTS[kind]
    x = synth.normal_bf16(m, k, 1.0, 51, 0)
    w = synth.normal_bf16(n, k, 0.02, 51, 1)
    xd = to_dev_bf16(x)
    packed = q.pack(q.quantize(to_dev_bf16(w), fmt))
    a = xd if kind == "w4a16" else q.quantize(xd, fmt)
    args = _gemm_args(a, packed, fmt, n, k)

    def pitched(dtype, pitch):
        buf = torch.full((m + 1, pitch), 77, dtype=dtype, device=DEV)
        q.linear(a, packed, fmt, n, out_dtype=q.QG_OUT_F32 if dtype == torch.float32 else q.QG_OUT_BF16, y=buf[:m, :n])
        torch.cuda.synchronize()
        assert bool((buf[m] == 77).all()) and bool((buf[:, n:] == 77).all())
        return buf[:m, :n]

    y = pitched(torch.float32, n)                       # staged
    rows = np.array([0, 255, 256, 287, 288, m - 1] * 6)
    cols = np.repeat(np.array([0, 191, 192, 255, 256, n - 1]), 6)
    check_linear(y, oracle.linear_reference(kind, x, w, rows, cols), rows, cols)
    for pitch in (n + 4, n + 1):                        # staged, element-wise
        assert torch.equal(pitched(torch.float32, pitch), y)
    for pitch in (n, n + 8, n + 2):                     # staged, staged, element-wise
        assert torch.equal(pitched(torch.bfloat16, pitch), y.bfloat16())

    s8 = (y.abs().max() / 448.0).reshape(1)
    want8 = (y * (1.0 / s8)).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    for pitch in (n, n + 16, n + 4, n + 1):             # staged, staged, element-wise (aligned dwords, bytes)
        buf = torch.full((m + 1, pitch), 77, dtype=torch.uint8, device=DEV)
        q.qg_gemm_quant(*args, buf, pitch, s8)
        torch.cuda.synchronize()
        assert torch.equal(buf[:m, :n], want8)
        assert bool((buf[m] == 77).all()) and bool((buf[:, n:] == 77).all())

    if kind == "w4a16":
        return                                          # no NVFP4 output for bf16 activations
    s4 = (y.abs().max() / 2688.0).reshape(1)
    codes, scales = oracle.quantize_nvfp4_static_f32(host(y), float(host(s4)[0]))
    for pitch in (-(-n // 128) * 128 + 128, n + 16):    # staged, element-wise
        cb = torch.full((m + 1, pitch // 2), 77, dtype=torch.uint8, device=DEV)
        sb = torch.full((m + 1, pitch // 16), 77, dtype=torch.uint8, device=DEV)
        q.qg_gemm_quant_nvfp4(*args, cb, sb, pitch, s4)
        torch.cuda.synchronize()
        assert np.array_equal(host(cb[:m, :n // 2]), codes) and np.array_equal(host(sb[:m, :n // 16]), scales)
        assert bool((cb[m] == 77).all()) and bool((cb[:, n // 2:] == 77).all())
        assert bool((sb[m] == 77).all()) and bool((sb[:, n // 16:] == 77).all())
