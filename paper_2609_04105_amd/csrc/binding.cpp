// Native call path of the Python binding: argument checks, output allocation and
// the C-ABI call of one forward or quantization in one step.
//
// Each function takes exactly the arguments of its Python wrapper (api.py), in
// order, and returns the result, or an int status other than FP4ATTN_OK, or None
// for any argument it does not take as it stands (another tensor class, device,
// layout, shape or type, a device that is not current): the wrapper then goes
// through its own checks, which accept or refuse the call.  Why native: a launch
// takes about 4 us, and the same checks in Python 7 us more (host time of a forward call
// 10.8 -> 4.0 us, of quantize_qkv 22.2 -> 8.5 us, of the smallest attention call 35.0 ->
// 12.9 us).
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <climits>

#include "../../include/fp4attn.h"

namespace {

using at::Tensor;

// A contiguous GPU tensor on the current device; nullptr otherwise.
const Tensor* gpu_tensor(PyObject* o, c10::DeviceIndex device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.get_device() != device || t.layout() != at::kStrided || !t.is_contiguous() || !t.has_storage())
    return nullptr;
  return &t;
}

bool is_shape(const Tensor& t, std::initializer_list<int64_t> s) {
  return t.sizes() == at::IntArrayRef(s.begin(), s.size());
}

// Plain floats, ints and bools only; anything else is left to Python.
bool as_float(PyObject* o, float* v) {
  if (PyFloat_CheckExact(o)) {
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
  }
  return false;
}
bool as_int(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x < INT_MIN || x > INT_MAX) return false;
  *v = (int32_t)x;
  return true;
}
bool as_bool(PyObject* o, bool* v) {
  *v = o == Py_True;
  return o == Py_True || o == Py_False;
}
bool as_dtype(PyObject* o, at::ScalarType* v) {
  if (!THPDtype_Check(o)) return false;
  *v = reinterpret_cast<THPDtype*>(o)->scalar_type;
  return *v == at::kFloat || *v == at::kBFloat16;
}
int c_dtype(at::ScalarType t) { return t == at::kBFloat16 ? FP4ATTN_BF16 : FP4ATTN_F32; }

void* stream_of(c10::DeviceIndex device) { return c10::hip::getCurrentHIPStream(device).stream(); }

Tensor gpu_empty(at::IntArrayRef shape, at::ScalarType type, c10::DeviceIndex device) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(at::Device(at::kCUDA, device)));
}

// Arguments of a forward that follow its operands.
struct ForwardArgs {
  float scale;
  fp4attn_forward_options opts;
  bool plain;  // no option given: the plain entry point
  Tensor out;
};

// softmax_scale, affine_a, affine_b, out, out_dtype, ex2_pairs, guard, causal, lse, pv_fp8
bool forward_args(PyObject* const* a, int64_t B, int64_t H, int64_t N, int64_t d, c10::DeviceIndex device,
                  ForwardArgs* f) {
  f->scale = (float)(1.0 / std::sqrt((double)d));
  if (a[0] != Py_None && !as_float(a[0], &f->scale)) return false;
  fp4attn_forward_options_init(&f->opts);
  if (!as_float(a[1], &f->opts.affine_a) || !as_float(a[2], &f->opts.affine_b)) return false;
  at::ScalarType type;
  if (!as_dtype(a[4], &type)) return false;
  if (a[5] != Py_None && !as_int(a[5], &f->opts.ex2_pairs)) return false;
  if (a[6] != Py_None) {
    if (!PyTuple_CheckExact(a[6]) || PyTuple_GET_SIZE(a[6]) != 2) return false;
    if (!as_int(PyTuple_GET_ITEM(a[6], 0), &f->opts.guard_margin) ||
        !as_int(PyTuple_GET_ITEM(a[6], 1), &f->opts.guard_shift))
      return false;
    f->opts.guard = 1;
  }
  bool causal, fp8;
  if (!as_bool(a[7], &causal) || !as_bool(a[9], &fp8)) return false;
  f->opts.causal = causal;
  f->opts.pv_fp8 = fp8;
  if (a[8] != Py_None) {
    const Tensor* lse = gpu_tensor(a[8], device);
    if (!lse || lse->scalar_type() != at::kFloat || !is_shape(*lse, {B, H, N})) return false;
    f->opts.lse = static_cast<float*>(lse->data_ptr());
  }
  f->plain = a[5] == Py_None && a[6] == Py_None && !causal && a[8] == Py_None && !fp8;
  if (a[3] != Py_None) {
    const Tensor* out = gpu_tensor(a[3], device);
    if (!out || (out->scalar_type() != at::kFloat && out->scalar_type() != at::kBFloat16) ||
        !is_shape(*out, {B, H, N, d}))
      return false;
    f->out = *out;
  } else {
    f->out = gpu_empty({B, H, N, d}, type, device);
  }
  return true;
}

int run_forward(const Tensor* const* ops, int64_t B, int64_t H, int64_t N, int64_t d, const ForwardArgs& f,
                c10::DeviceIndex device) {
  const uint8_t* p[6];
  for (int i = 0; i < 6; ++i) p[i] = static_cast<const uint8_t*>(ops[i]->data_ptr());
  void* out = f.out.data_ptr();
  const int type = c_dtype(f.out.scalar_type());
  void* stream = stream_of(device);
  int st;
  Py_BEGIN_ALLOW_THREADS
  if (f.plain)
    st = fp4attn_forward_mxfp4(p[0], p[1], p[2], p[3], p[4], p[5], B, H, N, d, f.scale, f.opts.affine_a,
                               f.opts.affine_b, out, type, stream);
  else
    st = fp4attn_forward_mxfp4_ex(p[0], p[1], p[2], p[3], p[4], p[5], B, H, N, d, f.scale, &f.opts, out, type, stream);
  Py_END_ALLOW_THREADS
  return st;
}

// Q, K and V of one shape, type and device, and their operands' tensors.
struct Qkv {
  const Tensor* x[3];
  Tensor ops[6];
};

bool qkv_args(PyObject* const* a, c10::DeviceIndex device, Qkv* r) {
  for (int i = 0; i < 3; ++i) {
    r->x[i] = gpu_tensor(a[i], device);
    if (!r->x[i]) return false;
  }
  const Tensor& q = *r->x[0];
  if (q.dim() < 2 || (q.scalar_type() != at::kFloat && q.scalar_type() != at::kBFloat16)) return false;
  for (int i = 1; i < 3; ++i)
    if (r->x[i]->scalar_type() != q.scalar_type() || r->x[i]->sizes() != q.sizes()) return false;
  return true;
}

int run_qkv(Qkv* r, bool anchored, bool fp8, c10::DeviceIndex device) {
  const Tensor& q = *r->x[0];
  const int64_t rows = q.size(-2), cols = q.size(-1);
  int64_t batch = 1;
  c10::SmallVector<int64_t, 6> shape(q.sizes().begin(), q.sizes().end());
  const size_t n = shape.size();
  for (size_t i = 0; i + 2 < n; ++i) batch *= shape[i];
  const int64_t dims[6][2] = {{rows, cols / 2}, {rows, cols / 32}, {rows, cols / 2}, {rows, cols / 32},
                              {cols, fp8 ? rows : rows / 2}, {cols, rows / 32}};
  uint8_t* p[6];
  for (int i = 0; i < 6; ++i) {
    shape[n - 2] = dims[i][0];
    shape[n - 1] = dims[i][1];
    r->ops[i] = gpu_empty(shape, at::kByte, device);
    p[i] = static_cast<uint8_t*>(r->ops[i].data_ptr());
  }
  const void *qp = q.data_ptr(), *kp = r->x[1]->data_ptr(), *vp = r->x[2]->data_ptr();
  const int type = c_dtype(q.scalar_type());
  void* stream = stream_of(device);
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = fp4attn_quantize_qkv(qp, kp, vp, type, batch, rows, cols, anchored ? 128 : 0, fp8, p[0], p[1], p[2], p[3], p[4],
                            p[5], stream);
  Py_END_ALLOW_THREADS
  return st;
}

// A C++ exception (a tensor without memory, an allocation that failed) leaves the
// call to Python, which meets the same condition and reports it as it always has.
template <class F>
PyObject* guarded(F&& f) {
  try {
    PyObject* r = f();
    if (r) return r;
  } catch (const std::exception&) {
  }
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// q_codes .. vt_scales, then forward_args
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 16) return nullptr;
    const c10::DeviceIndex device = c10::hip::current_device();
    const Tensor* ops[6];
    for (int i = 0; i < 6; ++i) {
      ops[i] = gpu_tensor(a[i], device);
      if (!ops[i] || ops[i]->scalar_type() != at::kByte || ops[i]->dim() != 4) return nullptr;
    }
    const auto s = ops[0]->sizes();
    const int64_t B = s[0], H = s[1], N = s[2], d = 2 * s[3];
    const int64_t vbytes = a[15] == Py_True ? N : N / 2;
    if (!is_shape(*ops[1], {B, H, N, d / 32}) || !is_shape(*ops[2], {B, H, N, d / 2}) ||
        !is_shape(*ops[3], {B, H, N, d / 32}) || !is_shape(*ops[4], {B, H, d, vbytes}) ||
        !is_shape(*ops[5], {B, H, d, N / 32}))
      return nullptr;
    ForwardArgs f;
    if (!forward_args(a + 6, B, H, N, d, device, &f)) return nullptr;
    const int st = run_forward(ops, B, H, N, d, f, device);
    if (st != FP4ATTN_OK) return PyLong_FromLong(st);
    if (a[9] != Py_None) {
      Py_INCREF(a[9]);
      return a[9];
    }
    return THPVariable_Wrap(std::move(f.out));
  });
}

// q, k, v, anchored, pv_fp8
PyObject* quantize_qkv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    bool anchored, fp8;
    if (n != 5 || !as_bool(a[3], &anchored) || !as_bool(a[4], &fp8) || (anchored && fp8)) return nullptr;
    const c10::DeviceIndex device = c10::hip::current_device();
    Qkv r;
    if (!qkv_args(a, device, &r)) return nullptr;
    const int st = run_qkv(&r, anchored, fp8, device);
    if (st != FP4ATTN_OK) return PyLong_FromLong(st);
    PyObject* t = PyTuple_New(6);
    for (int i = 0; t && i < 6; ++i) PyTuple_SET_ITEM(t, i, THPVariable_Wrap(std::move(r.ops[i])));
    return t;
  });
}

// q, k, v, then forward_args: quantization and forward
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 13) return nullptr;
    const c10::DeviceIndex device = c10::hip::current_device();
    Qkv r;
    if (!qkv_args(a, device, &r) || r.x[0]->dim() != 4) return nullptr;
    const auto s = r.x[0]->sizes();
    ForwardArgs f;
    if (s[2] % 32 != 0 || s[3] % 32 != 0 || !forward_args(a + 3, s[0], s[1], s[2], s[3], device, &f)) return nullptr;
    if (f.opts.guard && f.opts.pv_fp8) return nullptr;
    int st = run_qkv(&r, f.opts.guard != 0, f.opts.pv_fp8 != 0, device);
    const Tensor* ops[6];
    for (int i = 0; i < 6; ++i) ops[i] = &r.ops[i];
    if (st == FP4ATTN_OK) st = run_forward(ops, s[0], s[1], s[2], s[3], f, device);
    if (st != FP4ATTN_OK) return PyLong_FromLong(st);
    if (a[6] != Py_None) {
      Py_INCREF(a[6]);
      return a[6];
    }
    return THPVariable_Wrap(std::move(f.out));
  });
}

// q, k, v, softmax_scale, out, out_dtype
PyObject* forward_bf16(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 6) return nullptr;
    const c10::DeviceIndex device = c10::hip::current_device();
    Qkv r;
    if (!qkv_args(a, device, &r) || r.x[0]->dim() != 4 || r.x[0]->scalar_type() != at::kBFloat16) return nullptr;
    const auto s = r.x[0]->sizes();
    float scale = (float)(1.0 / std::sqrt((double)s[3]));
    at::ScalarType type;
    if ((a[3] != Py_None && !as_float(a[3], &scale)) || !as_dtype(a[5], &type)) return nullptr;
    Tensor out;
    if (a[4] != Py_None) {
      const Tensor* t = gpu_tensor(a[4], device);
      if (!t || (t->scalar_type() != at::kFloat && t->scalar_type() != at::kBFloat16) || t->sizes() != s) return nullptr;
      out = *t;
    } else {
      out = gpu_empty(s, type, device);
    }
    const void *qp = r.x[0]->data_ptr(), *kp = r.x[1]->data_ptr(), *vp = r.x[2]->data_ptr();
    void *op = out.data_ptr(), *stream = stream_of(device);
    const int ctype = c_dtype(out.scalar_type());
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = fp4attn_forward_bf16(qp, kp, vp, s[0], s[1], s[2], s[3], scale, op, ctype, stream);
    Py_END_ALLOW_THREADS
    if (st != FP4ATTN_OK) return PyLong_FromLong(st);
    if (a[4] != Py_None) {
      Py_INCREF(a[4]);
      return a[4];
    }
    return THPVariable_Wrap(std::move(out));
  });
}

PyMethodDef methods[] = {
    {"forward", (PyCFunction)(void (*)())forward, METH_FASTCALL, nullptr},
    {"quantize_qkv", (PyCFunction)(void (*)())quantize_qkv, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)())attention, METH_FASTCALL, nullptr},
    {"forward_bf16", (PyCFunction)(void (*)())forward_bf16, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module_def); }
