// torch_binding.cpp -- native form of the Python package's per-call helpers
// (quantize, linear, linear_fp8): argument checks, output allocation and the
// C-ABI call without a Python step in between. A linear's helper took 11 us of
// host time per call through ctypes (2 us per torch.empty, 3 us for the current
// stream, 4 us marshalling and launch) where the kernels of the small
// shapes take 3 to 6; this module takes 4 to 5.
//
// Each function handles the plain case (exact torch.Tensor arguments that
// pass every check of the Python helper) and returns None for anything else:
// the Python helper then goes on as if this module did not exist, and raises
// its own error where the arguments are wrong. A failed C-ABI call comes back
// as its status (an int). Allocation goes through the dispatcher (at::empty),
// and the GIL is released around it and the launch.
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "qgemm.h"

namespace {

struct Gil {  // released for a scope
  PyThreadState* s = PyEval_SaveThread();
  ~Gil() { PyEval_RestoreThread(s); }
};

PyObject* none() { Py_RETURN_NONE; }

// An exact torch.Tensor on the GPU, or null.
const at::Tensor* cuda_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() ? &t : nullptr;
}

bool int_of(PyObject* o, int64_t& v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  v = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}

// None: the current stream of the current device; an int: that handle.
bool stream_of(PyObject* o, void*& s) {
  if (o == Py_None) {
    s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  s = PyLong_AsVoidPtr(o);
  if (s == nullptr && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

bool rows_of_units(const at::Tensor& t) { return t.dim() == 2 && t.stride(1) == 1; }

bool dense2(const at::Tensor& t, int64_t r, int64_t c) {
  return t.scalar_type() == at::kByte && t.dim() == 2 && t.size(0) == r && t.size(1) == c && t.is_contiguous();
}

bool one_scale(const at::Tensor& t, const at::Device& dev) {
  return t.scalar_type() == at::kFloat && t.device() == dev && t.is_contiguous() && t.numel() >= 1;
}

bool packed_ok(const at::Tensor& t, const at::Device& dev) {
  return t.scalar_type() == at::kByte && t.device() == dev && t.is_contiguous();
}

at::Tensor empty2(int64_t r, int64_t c, at::ScalarType dt, const at::Device& dev) {
  return at::empty({r, c}, at::TensorOptions().dtype(dt).device(dev));
}

// quantize(x, fmt, stream, static_scale) -> (codes, block_scales, tensor_scale, rows, cols)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  const at::Tensor* xp = nargs == 4 ? cuda_tensor(a[0]) : nullptr;
  int64_t fmt;
  void* stream;
  if (!xp || !int_of(a[1], fmt) || !stream_of(a[2], stream)) return none();
  const at::Tensor& x = *xp;
  if (x.scalar_type() != at::kBFloat16 || !rows_of_units(x) || x.numel() == 0) return none();
  const int64_t rows = x.size(0), cols = x.size(1);
  const at::Device dev = x.device();
  const bool mx = fmt == QG_FMT_MXFP4 || fmt == QG_FMT_MXFP8;
  if (!(fmt == QG_FMT_FP8_E4M3 || (fmt == QG_FMT_NVFP4 && cols % 16 == 0) || (mx && cols % 32 == 0))) return none();
  const at::Tensor* sp = nullptr;
  if (a[3] != Py_None) {
    sp = cuda_tensor(a[3]);
    if (!sp || mx || !one_scale(*sp, dev)) return none();
  }
  at::Tensor codes, bs, ts;
  qg_status st;
  {
    Gil g;
    codes = empty2(rows, fmt == QG_FMT_FP8_E4M3 || fmt == QG_FMT_MXFP8 ? cols : cols / 2, at::kByte, dev);
    if (fmt != QG_FMT_FP8_E4M3) bs = empty2(rows, cols / (mx ? 32 : 16), at::kByte, dev);
    if (!mx && !sp) ts = at::empty({1}, at::TensorOptions().dtype(at::kFloat).device(dev));
    const int64_t ldx = rows > 1 ? x.stride(0) : cols;  // a size-1 dimension may carry any stride
    void* b = bs.defined() ? bs.data_ptr() : nullptr;
    if (sp)
      st = qg_quantize_act_static((qg_format)fmt, x.data_ptr(), rows, cols, ldx, codes.data_ptr(), b,
                                  static_cast<const float*>(sp->data_ptr()), stream);
    else
      st = qg_quantize_act((qg_format)fmt, x.data_ptr(), rows, cols, ldx, codes.data_ptr(), b,
                           ts.defined() ? static_cast<float*>(ts.data_ptr()) : nullptr, stream);
  }
  if (st != QG_OK) return PyLong_FromLong(st);
  PyObject* out = PyTuple_New(5);
  if (!out) return nullptr;
  auto put = [&](int i, const at::Tensor& t) {
    if (t.defined()) PyTuple_SET_ITEM(out, i, THPVariable_Wrap(t));
    else PyTuple_SET_ITEM(out, i, (Py_INCREF(Py_None), Py_None));
  };
  put(0, codes);
  put(1, bs);
  if (sp) PyTuple_SET_ITEM(out, 2, (Py_INCREF(a[3]), a[3]));
  else put(2, ts);
  PyTuple_SET_ITEM(out, 3, PyLong_FromLongLong(rows));
  PyTuple_SET_ITEM(out, 4, PyLong_FromLongLong(cols));
  return out;
  END_HANDLE_TH_ERRORS
}

// linear(a_fmt, data, block_scales, tensor_scale, rows, cols, w_packed, w_fmt, n, out_dtype, y, stream) -> y.
// a_fmt 0: data is the bf16 activation itself and rows, cols are ignored.
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  int64_t a_fmt, w_fmt, n, out;
  void* stream;
  const at::Tensor* dp = nargs == 12 ? cuda_tensor(a[1]) : nullptr;
  const at::Tensor* wp = dp ? cuda_tensor(a[6]) : nullptr;
  if (!wp || !int_of(a[0], a_fmt) || !int_of(a[7], w_fmt) || !int_of(a[8], n) || !int_of(a[9], out) ||
      !stream_of(a[11], stream))
    return none();
  const at::Tensor& d = *dp;
  const at::Device dev = d.device();
  if (!packed_ok(*wp, dev) || n < 0 || (out != QG_OUT_BF16 && out != QG_OUT_F32)) return none();
  int64_t m, k, lda;
  const at::Tensor *bs = nullptr, *ts = nullptr;
  if (a_fmt == QG_FMT_BF16) {
    if (d.scalar_type() != at::kBFloat16 || !rows_of_units(d)) return none();
    m = d.size(0);
    lda = k = d.size(1);
    if (m > 1) lda = d.stride(0);
  } else {
    if (!int_of(a[4], m) || !int_of(a[5], k) || m < 0 || k < 0) return none();
    lda = k;
    const bool mx = a_fmt == QG_FMT_MXFP4 || a_fmt == QG_FMT_MXFP8;
    if (a_fmt != QG_FMT_FP8_E4M3 && a_fmt != QG_FMT_NVFP4 && !mx) return none();
    if (!dense2(d, m, a_fmt == QG_FMT_FP8_E4M3 || a_fmt == QG_FMT_MXFP8 ? k : k / 2)) return none();
    if (a_fmt == QG_FMT_FP8_E4M3) {
      if (a[2] != Py_None) return none();
    } else {
      bs = cuda_tensor(a[2]);
      if (!bs || bs->device() != dev || !dense2(*bs, m, k / (mx ? 32 : 16))) return none();
    }
    if (mx) {
      if (a[3] != Py_None) return none();
    } else {
      ts = cuda_tensor(a[3]);
      if (!ts || !one_scale(*ts, dev)) return none();
    }
  }
  const at::ScalarType ydt = out == QG_OUT_F32 ? at::kFloat : at::kBFloat16;
  at::Tensor y;
  if (a[10] != Py_None) {
    const at::Tensor* yp = cuda_tensor(a[10]);
    if (!yp || yp->scalar_type() != ydt || yp->device() != dev || !rows_of_units(*yp) || yp->size(0) != m ||
        yp->size(1) != n)
      return none();
    y = *yp;
  }
  qg_status st;
  {
    Gil g;
    if (!y.defined()) y = empty2(m, n, ydt, dev);
    st = qg_gemm((qg_format)a_fmt, d.data_ptr(), bs ? bs->data_ptr() : nullptr,
                 ts ? static_cast<const float*>(ts->data_ptr()) : nullptr, lda, (qg_format)w_fmt, wp->data_ptr(),
                 (size_t)wp->numel(), m, n, k, y.data_ptr(), m > 1 ? y.stride(0) : n, (qg_out_dtype)out, stream);
  }
  if (st != QG_OK) return PyLong_FromLong(st);
  if (a[10] != Py_None) {
    Py_INCREF(a[10]);
    return a[10];
  }
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// linear_fp8(x, w_packed, n, out_dtype, stream) -> (y, tensor_scale)
PyObject* linear_fp8(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  int64_t n, out;
  void* stream;
  const at::Tensor* xp = nargs == 5 ? cuda_tensor(a[0]) : nullptr;
  const at::Tensor* wp = xp ? cuda_tensor(a[1]) : nullptr;
  if (!wp || !int_of(a[2], n) || !int_of(a[3], out) || !stream_of(a[4], stream)) return none();
  const at::Tensor& x = *xp;
  const at::Device dev = x.device();
  if (x.scalar_type() != at::kBFloat16 || !rows_of_units(x) || !packed_ok(*wp, dev) || n < 0 ||
      (out != QG_OUT_BF16 && out != QG_OUT_F32))
    return none();
  const int64_t m = x.size(0), k = x.size(1);
  at::Tensor y, ts;
  qg_status st;
  {
    Gil g;
    ts = at::empty({1}, at::TensorOptions().dtype(at::kFloat).device(dev));
    y = empty2(m, n, out == QG_OUT_F32 ? at::kFloat : at::kBFloat16, dev);
    st = qg_linear_fp8(x.data_ptr(), m > 1 ? x.stride(0) : k, static_cast<float*>(ts.data_ptr()), wp->data_ptr(),
                       (size_t)wp->numel(), m, n, k, y.data_ptr(), n, (qg_out_dtype)out, stream);
  }
  if (st != QG_OK) return PyLong_FromLong(st);
  PyObject* r = PyTuple_New(2);
  if (!r) return nullptr;
  PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(y));
  PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(ts));
  return r;
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"quantize", (PyCFunction)(void (*)())quantize, METH_FASTCALL, nullptr},
    {"linear", (PyCFunction)(void (*)())linear, METH_FASTCALL, nullptr},
    {"linear_fp8", (PyCFunction)(void (*)())linear_fp8, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qgemm_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qgemm_torch(void) { return PyModule_Create(&module); }
