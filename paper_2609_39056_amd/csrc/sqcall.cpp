// Native argument marshalling of the Python binding's hot calls.
//
// binding.py describes each call with ctypes structures, which costs 7-8 us of
// Python per linear (nine tensors checked one attribute at a time, two
// structures, ten converted arguments): more than the two kernels of a small
// layer take.  The functions here read the same tensors through torch's C++
// interface and call the C ABI entry whose address the binding passes, with the
// interpreter lock released as ctypes releases it.
//
// They only take the plain case: exact torch.Tensor objects on the GPU,
// contiguous, exact ActParams / Weight objects, ints.  For anything else
// they return NotImplemented and the binding goes on with its ctypes path,
// which accepts or refuses the arguments as it always has.  No C++ exception
// leaves them.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <exception>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "sq.h"

namespace {

PyObject* g_act_type = nullptr;     // binding.ActParams
PyObject* g_weight_type = nullptr;  // binding.Weight
PyObject* s_tok2stream;
PyObject* s_gamma;
PyObject* s_clip;
PyObject* s_dinv;
PyObject* s_step;
PyObject* s_range_mode;
PyObject* s_act_bits;
PyObject* s_qw;
PyObject* s_w_scale;
PyObject* s_bias;
PyObject* s_w_group;
PyObject* s_cuda_stream;

// The readers return whether the argument is plain.  They refuse without an
// exception: throwing one took 3-6 us, which a call that goes on to the ctypes
// path (13 us) would pay on top.

// An owned attribute of `o`; null, with a Python error set, if there is none.
struct Attr {
  PyObject* p;
  Attr(PyObject* o, PyObject* name) : p(PyObject_GetAttr(o, name)) {}
  ~Attr() { Py_XDECREF(p); }
  Attr(const Attr&) = delete;
  Attr& operator=(const Attr&) = delete;
};

const at::Tensor* tensor(PyObject* o) {
  if (o == nullptr || !THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

template <typename T>
bool read(PyObject* o, T*& p) {
  const at::Tensor* t = tensor(o);
  if (t == nullptr) return false;
  p = static_cast<T*>(t->data_ptr());
  return true;
}
template <typename T>
bool read_or_null(PyObject* o, T*& p) {
  p = nullptr;
  return o == Py_None || read(o, p);
}

// A buffer and its size.
bool read(PyObject* o, void*& p, size_t& bytes) {
  if (!read(o, p)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  bytes = static_cast<size_t>(t.numel()) * t.element_size();
  return true;
}
bool read_or_null(PyObject* o, void*& p, size_t& bytes) {
  p = nullptr;
  bytes = 0;
  return o == Py_None || read(o, p, bytes);
}

bool read_int(PyObject* o, int32_t& v) {
  if (o == nullptr || !PyLong_Check(o)) return false;
  const long w = PyLong_AsLong(o);
  v = static_cast<int32_t>(w);
  return w == v && !(w == -1 && PyErr_Occurred());
}

bool size32(int64_t w, int32_t& v) {
  v = static_cast<int32_t>(w);
  return w == v;
}

// A matrix and its number of rows.
template <typename T>
bool read_rows(PyObject* o, T*& p, int32_t& rows) {
  if (!read(o, p)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.dim() >= 1 && size32(t.size(0), rows);
}

bool read_stream(PyObject* o, hipStream_t& s) {
  if (o == Py_None) {
    s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  void* v;
  if (PyLong_CheckExact(o)) {
    v = PyLong_AsVoidPtr(o);
  } else {
    Attr a(o, s_cuda_stream);
    if (a.p == nullptr) return false;
    v = PyLong_AsVoidPtr(a.p);
  }
  s = static_cast<hipStream_t>(v);
  return v != nullptr || !PyErr_Occurred();
}

bool read(PyObject* o, sq_act_params& s) {
  if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_act_type) return false;
  Attr t2s(o, s_tok2stream), gamma(o, s_gamma), clip(o, s_clip), dinv(o, s_dinv), step(o, s_step),
      mode(o, s_range_mode), bits(o, s_act_bits);
  const at::Tensor* g = tensor(gamma.p);
  if (g == nullptr || g->dim() != 2) return false;
  s.gamma = static_cast<const float*>(g->data_ptr());
  return read_or_null(t2s.p, s.tok2stream) && read_or_null(clip.p, s.clip) && read_or_null(dinv.p, s.dinv) &&
         size32(g->size(1), s.num_streams) && size32(g->size(0), s.num_steps) && read_int(step.p, s.step) &&
         read_int(mode.p, s.range_mode) && read_int(bits.p, s.act_bits);
}

bool read(PyObject* o, sq_weight& s) {
  if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_weight_type) return false;
  Attr qw(o, s_qw), scale(o, s_w_scale), bias(o, s_bias), group(o, s_w_group);
  const at::Tensor* q = tensor(qw.p);
  if (q == nullptr || q->dim() < 2) return false;
  s.qw = static_cast<const uint8_t*>(q->data_ptr());
  return read_or_null(scale.p, s.w_scale) && read_or_null(bias.p, s.bias) && size32(q->size(0), s.N) &&
         size32(q->size(1) * 2, s.K) && read_int(group.p, s.w_group);
}

template <typename F>
bool read_entry(PyObject* address, F& fn) {
  void* p = PyLong_AsVoidPtr(address);
  fn = reinterpret_cast<F>(p);
  return p != nullptr;
}

// `args` reads the arguments (false: not plain; an exception of torch's counts as
// that), `call` makes the call.  The call runs without the interpreter lock and
// outside the try block: taking the lock back ends a daemon thread by a forced
// unwind once the interpreter shuts down, which no handler may catch (`...`
// would).
template <typename Args, typename Call>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, Args args, Call call) {
  if (n != want || g_act_type == nullptr) Py_RETURN_NOTIMPLEMENTED;
  bool plain = false;
  try {
    plain = args();
  } catch (const std::exception&) {
  }
  if (!plain) {
    PyErr_Clear();
    Py_RETURN_NOTIMPLEMENTED;
  }
  PyThreadState* save = PyEval_SaveThread();
  const sq_status st = call();
  PyEval_RestoreThread(save);
  return PyLong_FromLong(st);
}

// setup(ActParams, Weight)
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2) {
    PyErr_SetString(PyExc_TypeError, "setup(ActParams, Weight)");
    return nullptr;
  }
  Py_INCREF(a[0]);
  Py_INCREF(a[1]);
  Py_XDECREF(g_act_type);
  Py_XDECREF(g_weight_type);
  g_act_type = a[0];
  g_weight_type = a[1];
  Py_RETURN_NONE;
}

// linear(address, x, act, w, y, out_dtype, workspace, stream)
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_linear_w4a8) fn;
  sq_act_params act;
  sq_weight w;
  const uint16_t* x;
  int32_t M, out;
  void *y, *ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 8,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], x, M) && read(a[2], act) && read(a[3], w) && read(a[4], y) &&
               read_int(a[5], out) && read(a[6], ws, wb) && read_stream(a[7], s);
      },
      [&] { return fn(x, M, &act, &w, y, out, ws, wb, s); });
}

// gemm8(address, qx, row_scale, w, y, out_dtype, workspace, stream)
PyObject* gemm8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_gemm_w4a8) fn;
  sq_weight w;
  const int8_t* qx;
  const float* r;
  int32_t M, out;
  void *y, *ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 8,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], qx, M) && read(a[2], r) && read(a[3], w) && read(a[4], y) &&
               read_int(a[5], out) && read_or_null(a[6], ws, wb) && read_stream(a[7], s);
      },
      [&] { return fn(qx, r, M, &w, y, out, ws, wb, s); });
}

// gemm4(address, qx, group_scale, act, w, y, out_dtype, workspace, stream)
PyObject* gemm4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_gemm_w4a4) fn;
  sq_act_params act;
  sq_weight w;
  const uint8_t* qx;
  const uint16_t* g;
  int32_t M, out;
  void *y, *ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 9,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], qx, M) && read(a[2], g) && read(a[3], act) && read(a[4], w) &&
               read(a[5], y) && read_int(a[6], out) && read_or_null(a[7], ws, wb) && read_stream(a[8], s);
      },
      [&] { return fn(qx, g, M, &act, &w, y, out, ws, wb, s); });
}

// gemm4_fp8(address, qx, group_scale, kc, act, w, y, out_dtype, workspace, stream)
PyObject* gemm4_fp8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_gemm_w4a4_fp8) fn;
  sq_act_params act;
  sq_weight w;
  const uint8_t* qx;
  const float *g, *kc;
  int32_t M, out;
  void *y, *ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 10,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], qx, M) && read(a[2], g) && read(a[3], kc) && read(a[4], act) &&
               read(a[5], w) && read(a[6], y) && read_int(a[7], out) && read_or_null(a[8], ws, wb) &&
               read_stream(a[9], s);
      },
      [&] { return fn(qx, g, kc, M, &act, &w, y, out, ws, wb, s); });
}

// gelu8(address, x, act, w, act_next, qx_next, r_next, workspace, stream)
PyObject* gelu8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_linear_w4a8_gelu_quant) fn;
  sq_act_params act, next;
  sq_weight w;
  const uint16_t* x;
  int8_t* qx;
  float* r;
  int32_t M;
  void* ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 9,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], x, M) && read(a[2], act) && read(a[3], w) && read(a[4], next) &&
               read(a[5], qx) && read(a[6], r) && read(a[7], ws, wb) && read_stream(a[8], s);
      },
      [&] { return fn(x, M, &act, &w, &next, qx, r, ws, wb, s); });
}

// gelu4(address, x, act, w, act_next, qx_next, scale_next, kc_next, workspace, stream)
PyObject* gelu4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_linear_w4a4_gelu_quant) fn;
  sq_act_params act, next;
  sq_weight w;
  const uint16_t* x;
  float* kc;
  int32_t M;
  void *qx, *sc, *ws;
  size_t wb;
  hipStream_t s;
  return guarded(
      n, 10,
      [&] {
        return read_entry(a[0], fn) && read_rows(a[1], x, M) && read(a[2], act) && read(a[3], w) && read(a[4], next) &&
               read(a[5], qx) && read(a[6], sc) && read_or_null(a[7], kc) && read(a[8], ws, wb) &&
               read_stream(a[9], s);
      },
      [&] { return fn(x, M, &act, &w, &next, qx, sc, kc, ws, wb, s); });
}

// quantize(address, x, act, qx, act_scale, stream)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  decltype(&sq_quantize_act) fn;
  sq_act_params act;
  int32_t M, K;
  void *qx, *sc;
  hipStream_t s;
  const uint16_t* x;
  return guarded(
      n, 6,
      [&] {
        const at::Tensor* t = tensor(a[1]);
        return t != nullptr && t->dim() == 2 && size32(t->size(1), K) && read_entry(a[0], fn) &&
               read_rows(a[1], x, M) && read(a[2], act) && read(a[3], qx) && read(a[4], sc) && read_stream(a[5], s);
      },
      [&] { return fn(x, M, K, &act, qx, sc, s); });
}

PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(setup)), METH_FASTCALL, nullptr},
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
    {"gemm8", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gemm8)), METH_FASTCALL, nullptr},
    {"gemm4", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gemm4)), METH_FASTCALL, nullptr},
    {"gemm4_fp8", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gemm4_fp8)), METH_FASTCALL, nullptr},
    {"gelu8", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gelu8)), METH_FASTCALL, nullptr},
    {"gelu4", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gelu4)), METH_FASTCALL, nullptr},
    {"quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quantize)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "sqcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_sqcall(void) {
  s_tok2stream = PyUnicode_InternFromString("tok2stream");
  s_gamma = PyUnicode_InternFromString("gamma");
  s_clip = PyUnicode_InternFromString("clip");
  s_dinv = PyUnicode_InternFromString("dinv");
  s_step = PyUnicode_InternFromString("step");
  s_range_mode = PyUnicode_InternFromString("range_mode");
  s_act_bits = PyUnicode_InternFromString("act_bits");
  s_qw = PyUnicode_InternFromString("qw");
  s_w_scale = PyUnicode_InternFromString("w_scale");
  s_bias = PyUnicode_InternFromString("bias");
  s_w_group = PyUnicode_InternFromString("w_group");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  PyObject* m = PyModule_Create(&module_def);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", SQCALL_BUILT_FOR) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
