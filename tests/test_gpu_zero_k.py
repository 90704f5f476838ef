"""Linears whose K is zero: all outputs are zero, also where there are more of them
than a launch has threads (2^32)."""
import pytest
import torch

import paper_2609_21849_amd as q
from gpu_util import DEV, log

pytestmark = pytest.mark.gpu

FP8, NVFP4 = q.QG_FMT_FP8_E4M3, q.QG_FMT_NVFP4


def _packed(fmt, n):
    return torch.zeros(q.qg_packed_bytes(fmt, n, 0), dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("m,n", [(1, 16), (5, 272), (4100, 4112), (2 ** 20 + 1, 4096)])
def test_zero_k(m, n):
    log("k = 0, m=%d n=%d" % (m, n))
    s = torch.ones(1, device=DEV)
    w = _packed(FP8, n)
    y = torch.full((m + 1, n), 77, dtype=torch.uint8, device=DEV)
    q.qg_gemm_quant(FP8, None, None, s, 0, FP8, w, w.numel(), m, n, 0, y, n, s)
    assert not y[:m].any().item() and bool((y[m] == 77).all())
    del y
    y = torch.full((m + 1, n), 77, dtype=torch.bfloat16, device=DEV)
    q.qg_linear_fp8(torch.empty(16, dtype=torch.bfloat16, device=DEV), 0, torch.empty(1, device=DEV), w, w.numel(),
                    m, n, 0, y, n, q.QG_OUT_BF16)
    assert not y[:m].any().item() and bool((y[m] == 77).all())
    if m * n < 2 ** 32:
        y4 = torch.full((m + 1, n // 2), 77, dtype=torch.uint8, device=DEV)
        b4 = torch.full((m + 1, n // 16), 77, dtype=torch.uint8, device=DEV)
        w4 = _packed(NVFP4, n)
        q.qg_gemm_quant_nvfp4(NVFP4, None, None, s, 0, NVFP4, w4, w4.numel(), m, n, 0, y4, b4, n, s)
        for t in (y4, b4):
            assert not t[:m].any().item() and bool((t[m] == 77).all())
