"""The native per-call helpers against the Python statements they stand for:
every accepted form of the arguments gives the same tensors, whichever of the
two runs."""
import pytest
import torch

import paper_2609_21849_amd as q
import synth
from gpu_util import DEV, to_dev_bf16

pytestmark = pytest.mark.gpu


class _Off:
    """A native module that never takes a call."""
    quantize = linear = linear_fp8 = staticmethod(lambda *a: None)


def _both(monkeypatch, fn):
    native = fn()
    with monkeypatch.context() as mp:
        mp.setattr(q, "_host", _Off)
        python = fn()
    torch.cuda.synchronize()
    return native, python


def _same(a, b):
    if isinstance(a, q.QTensor):
        assert (a.fmt, a.rows, a.cols) == (b.fmt, b.rows, b.cols)
        a, b = (a.codes, a.block_scales, a.tensor_scale), (b.codes, b.block_scales, b.tensor_scale)
    if isinstance(a, tuple):
        assert len(a) == len(b)
        for u, v in zip(a, b):
            _same(u, v)
    elif a is None or b is None:
        assert a is b
    else:
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device
        assert torch.equal(a, b)


@pytest.mark.parametrize("rows", [0, 1, 9])
@pytest.mark.parametrize("fmt", [q.QG_FMT_FP8_E4M3, q.QG_FMT_NVFP4, q.QG_FMT_MXFP4, q.QG_FMT_MXFP8])
def test_quantize_forms(monkeypatch, fmt, rows):
    wide = to_dev_bf16(synth.normal_bf16(9, 640, 1.0, 3, 0))
    side = torch.cuda.Stream()
    scale = torch.full((1,), 2.0 ** -7, device=DEV)
    for x in (wide[:rows, :256].contiguous(), wide[:rows, 128:384]):
        _same(*_both(monkeypatch, lambda: q.quantize(x, fmt)))
        _same(*_both(monkeypatch, lambda: q.quantize(x, fmt, stream=torch.cuda.current_stream())))
        if fmt not in q.MX_FORMATS:
            a, b = _both(monkeypatch, lambda: q.quantize(x, fmt, static_scale=scale))
            _same(a, b)
            assert a.tensor_scale is scale
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):                   # the current stream, and its handle
            _same(*_both(monkeypatch, lambda: q.quantize(x, fmt)))
            _same(*_both(monkeypatch, lambda: q.quantize(x, fmt, stream=side.cuda_stream)))


@pytest.mark.parametrize("out", [q.QG_OUT_BF16, q.QG_OUT_F32])
@pytest.mark.parametrize("kind", ["fp8", "nvfp4", "mxfp4", "mxfp8", "w4a16", "fused"])
def test_linear_forms(monkeypatch, kind, out):
    fmt = {"fp8": 1, "fused": 1, "nvfp4": 2, "w4a16": 2, "mxfp4": 3, "mxfp8": 4}[kind]
    wide = to_dev_bf16(synth.normal_bf16(9, 640, 1.0, 3, 0))
    packed = q.pack(q.quantize(to_dev_bf16(synth.normal_bf16(48, 256, 0.02, 3, 1)), fmt))
    dt = torch.float32 if out == q.QG_OUT_F32 else torch.bfloat16
    for m in (0, 1, 9):
        for x in (wide[:m, :256].contiguous(), wide[:m, 128:384]):
            if kind == "fused":
                _same(*_both(monkeypatch, lambda: q.linear_fp8(x, packed, 48, out)))
                continue
            a = x if kind == "w4a16" else q.quantize(x, fmt)
            _same(*_both(monkeypatch, lambda: q.linear(a, packed, fmt, 48, out_dtype=out)))
            buf = torch.zeros((m, 64), dtype=dt, device=DEV)
            y, _ = _both(monkeypatch, lambda: q.linear(a, packed, fmt, 48, out_dtype=out, y=buf[:, :48]))
            assert torch.equal(y, q.linear(a, packed, fmt, 48, out_dtype=out)) and not buf[:, 48:].any()


def test_the_native_helpers_run():
    assert q._native().__name__ == "paper_2609_21849_amd._qgemm_torch"


def _late_input(op):
    """(the tensor that a producer fills late, its contents, the call)."""
    x = to_dev_bf16(synth.normal_bf16(64, 512, 1.0, 7, 0))
    if op.startswith("quantize"):
        fmt = q.QG_FMT_NVFP4 if op == "quantize nvfp4" else q.QG_FMT_FP8_E4M3
        return x, x.clone(), lambda **kw: q.quantize(x, fmt, **kw)
    wfmt = q.QG_FMT_NVFP4 if op == "linear w4a16" else q.QG_FMT_FP8_E4M3
    packed = q.pack(q.quantize(to_dev_bf16(synth.normal_bf16(256, 512, 0.02, 7, 1)), wfmt))
    if op == "linear_fp8":
        return x, x.clone(), lambda **kw: q.linear_fp8(x, packed, 256, **kw)
    if op == "linear w4a16":
        return x, x.clone(), lambda **kw: q.linear(x, packed, wfmt, 256, **kw)
    a = q.quantize(x, wfmt)
    return a.codes, a.codes.clone(), lambda **kw: q.linear(a, packed, wfmt, 256, **kw)


@pytest.mark.parametrize("op", ["quantize fp8", "quantize nvfp4", "linear fp8", "linear w4a16", "linear_fp8"])
@pytest.mark.parametrize("how", ["current", "handle", "stream"])
@pytest.mark.parametrize("native", [True, False])
def test_calls_run_on_the_stream_they_name(monkeypatch, op, how, native):
    """The input is filled on the side stream, behind some milliseconds of copies:
    a call that went to any other stream would read the zeros that are there
    before (the producer is still running when the call has returned)."""
    if not native:
        monkeypatch.setattr(q, "_host", _Off)
    late, value, call = _late_input(op)
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    work = torch.empty((2, 1 << 28), dtype=torch.float32, device=DEV)       # 1 GiB each
    work.zero_()
    want = call()
    torch.cuda.synchronize()
    for _ in range(2):                                  # the first also loads what runs
        late.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(24):
                work[0].copy_(work[1])
            late.copy_(value)
            done.record(side)
            if how == "current":
                got = call()
        if how == "handle":
            got = call(stream=side.cuda_stream)
        elif how == "stream":
            got = call(stream=side)
        running = not done.query()
        torch.cuda.synchronize()
        _same(got, want)
    assert running


def test_refusals_are_the_same(monkeypatch):
    x = to_dev_bf16(synth.normal_bf16(8, 256, 1.0, 5, 0))
    packed = q.pack(q.quantize(to_dev_bf16(synth.normal_bf16(32, 256, 0.02, 5, 1)), 1))
    a = q.quantize(x, 1)
    calls = [lambda: q.quantize(x[:, :24], 3), lambda: q.quantize(x, 9), lambda: q.quantize(x.t(), 1),
             lambda: q.quantize(x, 1, static_scale=torch.ones(1)), lambda: q.linear(a, packed, 1, 48),
             lambda: q.linear(a, packed, 2, 32), lambda: q.linear(x, packed, 1, 32), lambda: q.linear(a, packed[::2], 1, 32),
             lambda: q.linear(a, packed, 1, 32, out_dtype=5), lambda: q.linear_fp8(x[:, :64], packed, 32),
             lambda: q.linear_fp8(x.float(), packed, 32), lambda: q.linear_fp8(x, packed[:100], 32)]
    for fn in calls:
        errors = []
        for host in (None, _Off):
            with monkeypatch.context() as mp:
                if host is not None:
                    mp.setattr(q, "_host", host)
                with pytest.raises((ValueError, q.QGError)) as e:
                    fn()
            errors.append((type(e.value), str(e.value)))
        assert errors[0] == errors[1]
