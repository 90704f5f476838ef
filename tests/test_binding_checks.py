"""The Python binding refuses tensors in host memory before any library
call (the kernels would dereference their addresses on the GPU). Runs on the
CPU: every call below fails in the binding itself."""
import pytest
import torch

import paper_2609_21849_amd as q


def test_host_tensors_are_refused():
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="CUDA"):
        q.quantize(x, q.QG_FMT_FP8_E4M3)
    w = torch.zeros(4096, dtype=torch.uint8)
    with pytest.raises(ValueError, match="CUDA"):
        q.linear(x, w, q.QG_FMT_NVFP4, 16)
    with pytest.raises(ValueError, match="CUDA"):
        q.unpack(w, q.QG_FMT_FP8_E4M3, 16, 128)
    qt = q.QTensor(q.QG_FMT_FP8_E4M3, torch.zeros((4, 32), dtype=torch.uint8), None, torch.ones(1), 4, 32)
    with pytest.raises(ValueError, match="CUDA"):
        q.pack(qt)
    with pytest.raises(ValueError, match="CUDA"):
        q.dequantize(qt)
    # the one-to-one wrappers refuse host tensors too (raw int pointers pass as given)
    with pytest.raises(ValueError, match="CUDA"):
        q.qg_gemm(q.QG_FMT_BF16, x, None, None, 32, q.QG_FMT_NVFP4, w, w.numel(), 4, 16, 32, x, 16,
                  q.QG_OUT_BF16, stream=0)


def test_non_tensor_quantized_operand_is_refused():
    with pytest.raises(ValueError, match="QTensor"):
        q.dequantize(object())


def test_helpers_without_the_native_extension(monkeypatch):
    # libqgemm.so alone is enough: the Python statements take every call (and refuse what they always did)
    import sys
    monkeypatch.setitem(sys.modules, "paper_2609_21849_amd._qgemm_torch", None)  # importing it raises ImportError
    monkeypatch.delattr(q, "_qgemm_torch", raising=False)
    monkeypatch.setattr(q, "_host", None)
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    w = torch.zeros(4096, dtype=torch.uint8)
    with pytest.warns(RuntimeWarning, match="_qgemm_torch"), pytest.raises(ValueError, match="CUDA"):
        q.quantize(x, q.QG_FMT_FP8_E4M3)
    with pytest.raises(ValueError, match="CUDA"):
        q.linear(x, w, q.QG_FMT_NVFP4, 16)
    with pytest.raises(ValueError, match="CUDA"):
        q.linear_fp8(x, w, 16)


def test_arguments_are_checked_before_the_stream():
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    w = torch.zeros(4096, dtype=torch.uint8)
    for call in (lambda s: q.quantize(x, q.QG_FMT_FP8_E4M3, stream=s), lambda s: q.linear(x, w, q.QG_FMT_NVFP4, 16, stream=s),
                 lambda s: q.linear_fp8(x, w, 16, stream=s)):
        with pytest.raises(ValueError, match="CUDA"):
            call(object())


def test_build_without_a_host_compiler(monkeypatch, tmp_path, capsys):
    from paper_2609_21849_amd import build as b
    monkeypatch.setattr(b, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "libqgemm.so"))
    monkeypatch.setattr(b, "BINDING", str(tmp_path / "_qgemm_torch.so"))
    monkeypatch.setattr(b, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(b.shutil, "which", lambda name: None if name == "g++" else "/usr/bin/" + name)
    ran = []

    def run(cmd, **kw):
        ran.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return type("R", (), {"returncode": 0, "stderr": ""})()
    monkeypatch.setattr(b.subprocess, "run", run)
    (tmp_path / "_qgemm_torch.so").write_text("of another build")
    assert b.build() == b.LIB and len(ran) == 1  # the library's link alone
    assert (tmp_path / "libqgemm.so").exists() and not (tmp_path / "_qgemm_torch.so").exists()
    assert "no g++" in capsys.readouterr().err
