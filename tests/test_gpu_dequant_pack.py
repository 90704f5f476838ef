"""Dequantization by the hardware conversions and the one-launch pack / unpack,
against the oracle's tables and a plain statement of the packed layout: every
code with scales that make finite, overflowing, denormal and NaN products,
ragged ends and addresses off the vector alignment, and weights at the edges
of the 32-row panels and of the 128-byte column segments."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2609_21849_amd as q

pytestmark = pytest.mark.gpu

FP8, NV, M4, M8 = q.QG_FMT_FP8_E4M3, q.QG_FMT_NVFP4, q.QG_FMT_MXFP4, q.QG_FMT_MXFP8


def _bf16_bits(v):
    """RNE on the fp32 bits; NaN -> 0x7FC0 (the library's NaN)."""
    u = v.view(np.uint32).astype(np.uint64)
    r = (u + 0x7FFF + ((u >> 16) & 1)) >> 16
    return np.where(np.isnan(v), 0x7FC0, r).astype(np.uint16)


def _e4m3(codes):
    t = np.asarray(oracle.e4m3_table(), dtype=np.float32)
    assert t.shape == (256,)
    return t[codes]


def _bytes(n, shift, seed):
    rng = np.random.default_rng(seed)
    host = rng.integers(0, 256, n, dtype=np.uint8)
    buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
    buf[shift:shift + n] = torch.from_numpy(host).cuda()
    return host, buf[shift:shift + n]


def _dequant(fmt, codes, scales, ts, rows, cols, f32, shift=0):
    esz = 4 if f32 else 2
    out = torch.full((rows * cols * esz + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    o = out[shift:shift + rows * cols * esz]
    st = q.lib().qg_dequant(fmt, ctypes.c_void_p(codes.data_ptr()), ctypes.c_void_p(scales.data_ptr()) if scales is not None else None,
                           ctypes.c_void_p(ts.data_ptr()) if ts is not None else None, rows, cols,
                           ctypes.c_void_p(o.data_ptr()), q.QG_OUT_F32 if f32 else q.QG_OUT_BF16, None)
    assert st == 0
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert (got[:shift] == 0xAB).all() and (got[shift + rows * cols * esz:] == 0xAB).all()
    return got[shift:shift + rows * cols * esz].view(np.uint32 if f32 else np.uint16)


def _check(got, want, f32):
    if f32:
        nan = np.isnan(want)
        assert np.array_equal(np.isnan(got.view(np.float32)), nan)
        assert np.array_equal(got[~nan], want.view(np.uint32)[~nan])
    else:
        assert np.array_equal(got, _bf16_bits(want))


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("rows,cols,shift", [(1, 1, 0), (1, 15, 0), (3, 257, 0), (16, 256, 0), (16, 256, 4), (5, 1000, 0)])
@pytest.mark.parametrize("scale", [0.0, 1.0, 0.0123, 1e-40, 1e37, float("inf"), float("nan")])
def test_fp8_dequant_bits(rows, cols, shift, scale, f32):
    host, codes = _bytes(rows * cols, shift, rows * cols)
    if cols == 256:  # clean rows too: the fast path beside the NaN codes
        host[: 8 * 256] = np.arange(8 * 256, dtype=np.uint8) % 127
        codes[: 8 * 256] = torch.from_numpy(host[: 8 * 256]).cuda()
    with np.errstate(all="ignore"):
        want = _e4m3(host) * np.float32(scale)
    _check(_dequant(FP8, codes, None, torch.tensor([scale], device="cuda"), rows, cols, f32, shift), want, f32)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("rows,cols,cshift,oshift", [(1, 16, 0, 0), (1, 16 * 256, 8, 0), (33, 16 * 33, 0, 4)])
@pytest.mark.parametrize("scale", [1.0, 0.0123, 1e-40, 3e37, float("inf"), float("nan")])
def test_nvfp4_dequant_bits(rows, cols, cshift, oshift, scale, f32):
    n = rows * cols
    host, codes = _bytes(n // 2, cshift, n)
    sb, scales = _bytes(n // 16, 1, n + 1)
    if n // 16 == 256:
        sb[:] = np.arange(256)
        scales.copy_(torch.from_numpy(sb).cuda())
    e = np.asarray(oracle.e2m1_table(), dtype=np.float32)[np.stack([host & 15, host >> 4], 1).reshape(-1)]
    with np.errstate(all="ignore"):
        want = (e * np.repeat(_e4m3(sb), 16)) * np.float32(scale)
    _check(_dequant(NV, codes, scales, torch.tensor([scale], device="cuda"), rows, cols, f32, oshift), want, f32)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("fmt,shift", [(M4, 0), (M4, 4), (M8, 0), (M8, 8)])
def test_mx_dequant_bits(fmt, shift, f32):
    rows, cols = 4, 32 * 80
    n = rows * cols
    host, codes = _bytes(n // 2 if fmt == M4 else n, shift, 5)
    sc, scales = _bytes(n // 32, 3, 6)
    sc[:256] = np.arange(256)
    scales.copy_(torch.from_numpy(sc).cuda())
    e = (np.asarray(oracle.e2m1_table(), dtype=np.float32)[np.stack([host & 15, host >> 4], 1).reshape(-1)]
         if fmt == M4 else _e4m3(host))
    with np.errstate(all="ignore"):
        s = np.where(sc == 255, np.nan, np.ldexp(1.0, sc.astype(np.int64) - 127)).astype(np.float32)
        want = e * np.repeat(s, 32)
    _check(_dequant(fmt, codes, scales, None, rows, cols, f32), want, f32)


def _packed_codes(fmt, canon, n, k):
    """The layout as stated in csrc/pack.hip, piece by piece of 16 bytes."""
    p = (n + 31) // 32
    rb = k if fmt in (FP8, M8) else k // 2
    c = np.zeros((p * 32, rb), np.uint8)
    c[:n] = canon.reshape(n, rb)
    c = c.reshape(p, 32, rb // 16, 16)
    if fmt == FP8:  # pieces (chunk, t, g, h) -> images (chunk, t, h)[g][row]
        v = c.reshape(p, 32, rb // 128, 2, 2, 2, 16).transpose(0, 2, 3, 5, 4, 1, 6)
    elif fmt == M8:  # pieces (chunk, t, h, g) -> images (chunk, t, h)[g][row]
        v = c.reshape(p, 32, rb // 128, 2, 2, 2, 16).transpose(0, 2, 3, 4, 5, 1, 6)
    elif fmt == NV:  # pieces (chunk, g, h) -> images (chunk, h)[g][row]
        v = c.reshape(p, 32, rb // 64, 2, 2, 16).transpose(0, 2, 4, 3, 1, 5)
    else:  # pieces (step, g) -> images (step)[g][row]
        v = c.reshape(p, 32, rb // 32, 2, 16).transpose(0, 2, 3, 1, 4)
    return np.ascontiguousarray(v).reshape(-1)


def _packed_scales(fmt, canon, n, k):
    p = (n + 31) // 32
    if fmt == NV:
        c = np.zeros((p * 32, k // 16), np.uint8)
        c[:n] = canon.reshape(n, k // 16)
        return np.ascontiguousarray(c.reshape(p, 32, k // 128, 8).transpose(0, 2, 1, 3)).reshape(-1)
    c = np.zeros((p * 32, k // 32), np.uint8)
    c[:n] = canon.reshape(n, k // 32)
    return np.ascontiguousarray(c.reshape(p, 32, k // 256, 4, 2).transpose(0, 2, 4, 1, 3)).reshape(-1)


@pytest.mark.parametrize("fmt", [FP8, NV, M4, M8])
@pytest.mark.parametrize("n,k", [(16, 256), (32, 384), (48, 128), (80, 1280), (2080, 768)])
def test_pack_layout_and_round_trip(fmt, n, k):
    if fmt in (M4, M8) and k % 256:
        k += 128
    rb = k if fmt in (FP8, M8) else k // 2
    host, codes = _bytes(n * rb, 0, n + k)
    sc_host = scales = None
    if fmt != FP8:
        sc_host, scales = _bytes(n * k // (16 if fmt == NV else 32), 0, n + k + 1)
    ts = torch.tensor([0.375], device="cuda") if fmt in (FP8, NV) else None
    packed = q.pack(q.QTensor(fmt, codes.reshape(n, rb), None if scales is None else scales.reshape(n, -1), ts, n, k))
    got = packed.cpu().numpy()
    want = _packed_codes(fmt, host, n, k)
    assert np.array_equal(got[256:256 + want.size], want)
    if fmt != FP8:
        ws = _packed_scales(fmt, sc_host, n, k)
        assert np.array_equal(got[256 + want.size:256 + want.size + ws.size], ws)
    assert got[:8].view(np.uint32).tolist() == [0x57504751, 3] and got[16:32].view(np.int64).tolist() == [n, k]
    assert got[8:16].view(np.uint32).tolist() == [fmt, 0]
    assert got[32:36].view(np.float32)[0] == (0.375 if ts is not None else 1.0)
    back = q.unpack(packed, fmt, n, k)
    assert np.array_equal(back.codes.cpu().numpy().reshape(-1), host)
    if fmt != FP8:
        assert np.array_equal(back.block_scales.cpu().numpy().reshape(-1), sc_host)
    if ts is not None:
        assert back.tensor_scale.item() == 0.375
