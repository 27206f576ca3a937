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
// contiguous, exact ActParams / Weight objects, plain ints.  For anything else
// they return NotImplemented and the binding goes on with its ctypes path,
// which accepts or refuses the arguments as it always has.  No C++ exception
// leaves them.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <exception>
#include <optional>

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

struct NotPlain {};  // thrown and caught inside this file

// An owned attribute of `o`.
struct Attr {
  PyObject* p;
  Attr(PyObject* o, PyObject* name) : p(PyObject_GetAttr(o, name)) {
    if (p == nullptr) throw NotPlain{};
  }
  ~Attr() { Py_DECREF(p); }
  Attr(const Attr&) = delete;
  Attr& operator=(const Attr&) = delete;
};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain{};
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) throw NotPlain{};
  return t;
}

void* ptr(PyObject* o) { return tensor(o).data_ptr(); }
void* ptr_or_null(PyObject* o) { return o == Py_None ? nullptr : ptr(o); }

int32_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw NotPlain{};
  const long v = PyLong_AsLong(o);
  if (v != static_cast<int32_t>(v)) throw NotPlain{};  // also an overflow's -1 with an error set
  if (v == -1 && PyErr_Occurred()) throw NotPlain{};
  return static_cast<int32_t>(v);
}

int32_t size32(int64_t v) {
  if (v != static_cast<int32_t>(v)) throw NotPlain{};
  return static_cast<int32_t>(v);
}

int32_t rows(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.dim() < 1) throw NotPlain{};
  return size32(t.size(0));
}

size_t bytes(PyObject* o) {
  const at::Tensor& t = tensor(o);
  return static_cast<size_t>(t.numel()) * t.element_size();
}
size_t bytes_or_zero(PyObject* o) { return o == Py_None ? 0 : bytes(o); }

hipStream_t stream(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  if (PyLong_CheckExact(o)) {
    void* v = PyLong_AsVoidPtr(o);
    if (v == nullptr && PyErr_Occurred()) throw NotPlain{};
    return static_cast<hipStream_t>(v);
  }
  Attr a(o, s_cuda_stream);
  void* v = PyLong_AsVoidPtr(a.p);
  if (v == nullptr && PyErr_Occurred()) throw NotPlain{};
  return static_cast<hipStream_t>(v);
}

struct Act {
  sq_act_params s;
  explicit Act(PyObject* o) {
    if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_act_type) throw NotPlain{};
    Attr t2s(o, s_tok2stream), gamma(o, s_gamma), clip(o, s_clip), dinv(o, s_dinv), step(o, s_step),
        mode(o, s_range_mode), bits(o, s_act_bits);
    const at::Tensor& g = tensor(gamma.p);
    if (g.dim() != 2) throw NotPlain{};
    s.tok2stream = static_cast<const int32_t*>(ptr_or_null(t2s.p));
    s.gamma = static_cast<const float*>(g.data_ptr());
    s.clip = static_cast<const float*>(ptr_or_null(clip.p));
    s.dinv = static_cast<const float*>(ptr_or_null(dinv.p));
    s.num_streams = size32(g.size(1));
    s.num_steps = size32(g.size(0));
    s.step = integer(step.p);
    s.range_mode = integer(mode.p);
    s.act_bits = integer(bits.p);
  }
};

struct Weight {
  sq_weight s;
  explicit Weight(PyObject* o) {
    if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_weight_type) throw NotPlain{};
    Attr qw(o, s_qw), scale(o, s_w_scale), bias(o, s_bias), group(o, s_w_group);
    const at::Tensor& q = tensor(qw.p);
    if (q.dim() < 2) throw NotPlain{};
    s.qw = static_cast<const uint8_t*>(q.data_ptr());
    s.w_scale = static_cast<const uint16_t*>(ptr_or_null(scale.p));
    s.bias = static_cast<const uint16_t*>(ptr_or_null(bias.p));
    s.N = size32(q.size(0));
    s.K = size32(q.size(1) * 2);
    s.w_group = integer(group.p);
  }
};

template <typename F>
F entry(PyObject* address) {
  void* p = PyLong_AsVoidPtr(address);
  if (p == nullptr) throw NotPlain{};
  return reinterpret_cast<F>(p);
}

// `prepare` reads the arguments and returns the call to make.  Everything that is
// not plain, C++ exceptions of torch included, becomes NotImplemented.  The call
// itself runs without the interpreter lock and outside the try block: taking the
// lock back ends a daemon thread by a forced unwind once the interpreter shuts
// down, which no handler may catch (`...` would).
template <typename Prepare>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, Prepare prepare) {
  if (n != want || g_act_type == nullptr) Py_RETURN_NOTIMPLEMENTED;
  std::optional<decltype(prepare())> call;
  try {
    call.emplace(prepare());
  } catch (const NotPlain&) {
  } catch (const std::exception&) {
  }
  if (!call) {
    PyErr_Clear();
    Py_RETURN_NOTIMPLEMENTED;
  }
  PyThreadState* save = PyEval_SaveThread();
  const sq_status st = (*call)();
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
  return guarded(n, 8, [&] {
    const auto fn = entry<decltype(&sq_linear_w4a8)>(a[0]);
    const Act act(a[2]);
    const Weight w(a[3]);
    const uint16_t* x = static_cast<const uint16_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]), out = integer(a[5]);
    void* y = ptr(a[4]);
    void* ws = ptr(a[6]);
    const size_t wb = bytes(a[6]);
    const hipStream_t s = stream(a[7]);
    return [=] { return fn(x, M, &act.s, &w.s, y, out, ws, wb, s); };
  });
}

// gemm8(address, qx, row_scale, w, y, out_dtype, workspace, stream)
PyObject* gemm8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&] {
    const auto fn = entry<decltype(&sq_gemm_w4a8)>(a[0]);
    const Weight w(a[3]);
    const int8_t* qx = static_cast<const int8_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]), out = integer(a[5]);
    const float* r = static_cast<const float*>(ptr(a[2]));
    void* y = ptr(a[4]);
    void* ws = ptr_or_null(a[6]);
    const size_t wb = bytes_or_zero(a[6]);
    const hipStream_t s = stream(a[7]);
    return [=] { return fn(qx, r, M, &w.s, y, out, ws, wb, s); };
  });
}

// gemm4(address, qx, group_scale, act, w, y, out_dtype, workspace, stream)
PyObject* gemm4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&] {
    const auto fn = entry<decltype(&sq_gemm_w4a4)>(a[0]);
    const Act act(a[3]);
    const Weight w(a[4]);
    const uint8_t* qx = static_cast<const uint8_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]), out = integer(a[6]);
    const uint16_t* g = static_cast<const uint16_t*>(ptr(a[2]));
    void* y = ptr(a[5]);
    void* ws = ptr_or_null(a[7]);
    const size_t wb = bytes_or_zero(a[7]);
    const hipStream_t s = stream(a[8]);
    return [=] { return fn(qx, g, M, &act.s, &w.s, y, out, ws, wb, s); };
  });
}

// gemm4_fp8(address, qx, group_scale, kc, act, w, y, out_dtype, workspace, stream)
PyObject* gemm4_fp8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    const auto fn = entry<decltype(&sq_gemm_w4a4_fp8)>(a[0]);
    const Act act(a[4]);
    const Weight w(a[5]);
    const uint8_t* qx = static_cast<const uint8_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]), out = integer(a[7]);
    const float* g = static_cast<const float*>(ptr(a[2]));
    const float* kc = static_cast<const float*>(ptr(a[3]));
    void* y = ptr(a[6]);
    void* ws = ptr_or_null(a[8]);
    const size_t wb = bytes_or_zero(a[8]);
    const hipStream_t s = stream(a[9]);
    return [=] { return fn(qx, g, kc, M, &act.s, &w.s, y, out, ws, wb, s); };
  });
}

// gelu8(address, x, act, w, act_next, qx_next, r_next, workspace, stream)
PyObject* gelu8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&] {
    const auto fn = entry<decltype(&sq_linear_w4a8_gelu_quant)>(a[0]);
    const Act act(a[2]), next(a[4]);
    const Weight w(a[3]);
    const uint16_t* x = static_cast<const uint16_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]);
    int8_t* qx = static_cast<int8_t*>(ptr(a[5]));
    float* r = static_cast<float*>(ptr(a[6]));
    void* ws = ptr(a[7]);
    const size_t wb = bytes(a[7]);
    const hipStream_t s = stream(a[8]);
    return [=] { return fn(x, M, &act.s, &w.s, &next.s, qx, r, ws, wb, s); };
  });
}

// gelu4(address, x, act, w, act_next, qx_next, scale_next, kc_next, workspace, stream)
PyObject* gelu4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    const auto fn = entry<decltype(&sq_linear_w4a4_gelu_quant)>(a[0]);
    const Act act(a[2]), next(a[4]);
    const Weight w(a[3]);
    const uint16_t* x = static_cast<const uint16_t*>(ptr(a[1]));
    const int32_t M = rows(a[1]);
    void* qx = ptr(a[5]);
    void* sc = ptr(a[6]);
    float* kc = static_cast<float*>(ptr_or_null(a[7]));
    void* ws = ptr(a[8]);
    const size_t wb = bytes(a[8]);
    const hipStream_t s = stream(a[9]);
    return [=] { return fn(x, M, &act.s, &w.s, &next.s, qx, sc, kc, ws, wb, s); };
  });
}

// quantize(address, x, act, qx, act_scale, stream)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&] {
    const auto fn = entry<decltype(&sq_quantize_act)>(a[0]);
    const at::Tensor& x = tensor(a[1]);
    if (x.dim() != 2) throw NotPlain{};
    const Act act(a[2]);
    const int32_t M = size32(x.size(0)), K = size32(x.size(1));
    const uint16_t* xp = static_cast<const uint16_t*>(x.data_ptr());
    void* qx = ptr(a[3]);
    void* sc = ptr(a[4]);
    const hipStream_t s = stream(a[5]);
    return [=] { return fn(xp, M, K, &act.s, qx, sc, s); };
  });
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
