// The calls of a training or inference step, from Python tensors to the C entry points.  On small graphs a step's time is the host's:
// a GCN layer of 4096 vertices is five calls and six launches that the GPU ends in 20.4 us; each call spent 1.9 us in Python and ctypes
// beside some 2.7 us a launch, 26.2 us in all, and spends 0.28 here, 18.8 in all (0.2 more with a stream object).
//
// A function takes what its Python wrapper takes, in the wrapper's order, and returns the call's status, or -1 (kOther) without having
// called anything when an argument is not of the plain form (a tensor of the expected type on the GPU, an int, a float, a stream, None where
// that is allowed): the wrapper then goes its own way, which takes all other forms and raises what is to be raised.  Nothing is kept between
// calls but the addresses of the entry points, which bind() takes from the loaded library.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/core/Tensor.h>

#include <climits>
#include <cstdint>
#include <cstring>
#include <exception>
#include <new>
#include <optional>

#include "hgnn.h"

namespace {

constexpr long kOther = -1;

PyObject *g_raw_stream = nullptr, *g_current_device = nullptr;  // torch's functions: the current stream of a device as a number, the current device
PyObject *g_struct = nullptr, *g_handle = nullptr, *g_cuda_stream = nullptr;  // attribute names

struct Table {  // a vertex-level tensor: rows of a pitch, unit stride along the features
  void* p = nullptr;
  int64_t ld = 0, rows = 0, cols = 0;
  hgnn_half* half() const { return static_cast<hgnn_half*>(p); }
  float* single() const { return static_cast<float*>(p); }
};

// Reads arguments; ok turns false with the first that is not plain.
struct Reader {
  bool ok = true;

  const at::Tensor* tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) {  // (a parameter is plain, another subclass is not)
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda()) {
      ok = false;
      return nullptr;
    }
    return &t;
  }
  void* data(PyObject* o, at::ScalarType type) {
    const at::Tensor* const t = tensor(o);
    if (!t) return nullptr;
    if (t->scalar_type() != type) {
      ok = false;
      return nullptr;
    }
    return t->data_ptr();
  }
  void* data_or_null(PyObject* o, at::ScalarType type) { return o == Py_None ? nullptr : data(o, type); }
  hgnn_half* half(PyObject* o) { return static_cast<hgnn_half*>(data(o, at::kHalf)); }
  hgnn_half* half_or_null(PyObject* o) { return static_cast<hgnn_half*>(data_or_null(o, at::kHalf)); }
  float* single(PyObject* o) { return static_cast<float*>(data(o, at::kFloat)); }
  float* single_or_null(PyObject* o) { return static_cast<float*>(data_or_null(o, at::kFloat)); }
  Table table(PyObject* o, at::ScalarType type = at::kHalf) {
    Table r;
    r.p = data(o, type);
    if (!ok) return r;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.dim() != 2 || t.stride(1) != 1) {
      ok = false;
      return r;
    }
    r.ld = t.stride(0), r.rows = t.size(0), r.cols = t.size(1);
    return r;
  }
  Table table_or_null(PyObject* o) { return o == Py_None ? Table() : table(o); }
  void* workspace(PyObject* o, size_t* bytes) {
    *bytes = 0;
    const at::Tensor* const t = tensor(o);
    if (!t) return nullptr;
    *bytes = size_t(t->numel()) * size_t(t->element_size());
    return t->data_ptr();
  }
  int integer(PyObject* o) {
    if (!PyLong_Check(o)) {
      ok = false;
      return 0;
    }
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT_MIN || v > INT_MAX) ok = false;
    return int(v);
  }
  int integer_or(PyObject* o, int64_t otherwise) {
    if (o != Py_None) return integer(o);
    if (otherwise > INT_MAX) ok = false;
    return int(otherwise);
  }
  float real(PyObject* o) {  // (an int is one, as to ctypes)
    if (PyFloat_Check(o)) return float(PyFloat_AS_DOUBLE(o));
    if (!PyLong_Check(o)) {
      ok = false;
      return 0.f;
    }
    return float(PyLong_AsDouble(o));
  }
  bool truth(PyObject* o) {  // of a bool or another int
    if (PyLong_Check(o)) return PyObject_IsTrue(o) == 1;
    ok = false;
    return false;
  }
  hgnn_csr graph(PyObject* o) {  // a copy of the structure inside a Csr, which is anybody's while the lock is not held
    hgnn_csr g{};
    PyObject* const s = PyObject_GetAttr(o, g_struct);
    Py_buffer b;
    if (!s || PyObject_GetBuffer(s, &b, PyBUF_SIMPLE) != 0) {
      Py_XDECREF(s);
      ok = false;
      return g;
    }
    if (size_t(b.len) == sizeof(g)) std::memcpy(&g, b.buf, sizeof(g));
    else ok = false;
    PyBuffer_Release(&b);
    Py_DECREF(s);
    return g;
  }
  hgnn_plan* plan(PyObject* o) {  // of a Plan that has not been destroyed
    PyObject* const h = PyObject_GetAttr(o, g_handle);
    void* const p = h && PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
    Py_XDECREF(h);
    if (!p) ok = false;
    return static_cast<hgnn_plan*>(p);
  }
  hgnn_plan* plan_or_null(PyObject* o) { return o == Py_None ? nullptr : plan(o); }
  void* stream(PyObject* o) {  // None: the current one; a number, or what has one as its cuda_stream
    if (o != Py_None) {
      if (PyLong_CheckExact(o)) return PyLong_AsVoidPtr(o);
      PyObject* const raw = PyObject_GetAttr(o, g_cuda_stream);
      void* const s = raw && PyLong_CheckExact(raw) ? PyLong_AsVoidPtr(raw) : nullptr;
      if (!raw || !PyLong_CheckExact(raw)) ok = false;
      Py_XDECREF(raw);
      return s;
    }
    PyObject* const device = PyObject_CallNoArgs(g_current_device);
    PyObject* const raw = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    void* const s = raw ? PyLong_AsVoidPtr(raw) : nullptr;
    if (!raw) ok = false;
    Py_XDECREF(device);
    Py_XDECREF(raw);
    return s;
  }
};

// f(reader, arguments) reads them and returns what calls the entry point; that runs without the interpreter's lock.  An exception of the library's becomes
// one of Python's once the lock is held again: the call has been made and is not repeated.  Nothing is caught around taking the lock, where a thread that
// outlives the interpreter is unwound.
template <class F>
PyObject* run(PyObject* const* a, Py_ssize_t n, Py_ssize_t want, F&& f) {
  long status = kOther;
  if (n == want && g_raw_stream) {
    Reader r;
    std::optional<decltype(f(r, a))> call;
    try {
      call.emplace(f(r, a));
    } catch (const std::exception&) {  // a tensor without memory of its own: the wrapper raises what torch says of it
    }
    const bool plain = call && r.ok && !PyErr_Occurred();
    PyErr_Clear();
    if (plain) {
      PyObject* failed = nullptr;
      char what[256] = "";
      Py_BEGIN_ALLOW_THREADS
      try {
        status = long((*call)());
      } catch (const std::bad_alloc&) {
        failed = PyExc_MemoryError;
      } catch (const std::exception& e) {
        failed = PyExc_RuntimeError;
        std::strncpy(what, e.what(), sizeof(what) - 1);
      }
      Py_END_ALLOW_THREADS
      if (failed) {
        PyErr_SetString(failed, what);
        return nullptr;
      }
    }
  }
  return PyLong_FromLong(status);
}

#define HGNN_ENTRIES(X)                                                                                                          \
  X(linear) X(linear_padded) X(linear_wgrad) X(spmm) X(spmm_discretized) X(spmm_discretized_fused) X(sddmm) X(edge_softmax)       \
  X(edge_softmax_bwd) X(edge_rowsum) X(edge_colsum) X(gat_forward_fused) X(gat_forward_fused_save) X(gat_backward_fused_saved) \
  X(gat_feature_grad)
#define HGNN_ENTRY(name) decltype(&hgnn_##name) f_##name = nullptr;
HGNN_ENTRIES(HGNN_ENTRY)

#define HGNN_CALL(name, count) PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t n) { return run(args, n, count, [](Reader& r, PyObject* const* a)
#define HGNN_END ); }

HGNN_CALL(linear, 7) {
  const Table X = r.table(a[0]), W = r.table(a[1]), Y = r.table(a[2]);
  const bool trans = r.truth(a[3]);
  const int K = r.integer_or(a[4], X.cols), F = r.integer_or(a[5], trans ? W.rows : W.cols);
  void* const s = r.stream(a[6]);
  const int64_t KW = trans ? K : W.rows;
  return [=] {
    if (KW < K) return f_linear_padded(X.rows, K, int(KW), F, X.half(), X.ld, W.half(), W.ld, Y.half(), Y.ld, s);
    return f_linear(X.rows, K, F, X.half(), X.ld, W.half(), W.ld, trans, Y.half(), Y.ld, s);
  };
} HGNN_END

HGNN_CALL(linear_wgrad, 7) {
  const Table X = r.table(a[0]), dY = r.table(a[1]), dW = r.table(a[2], at::kFloat);
  size_t bytes;
  void* const ws = r.workspace(a[3], &bytes);
  const int K = r.integer_or(a[4], X.cols), F = r.integer_or(a[5], dY.cols);
  void* const s = r.stream(a[6]);
  return [=] { return f_linear_wgrad(X.rows, K, F, X.half(), X.ld, dY.half(), dY.ld, dW.single(), dW.ld, ws, bytes, s); };
} HGNN_END

HGNN_CALL(spmm, 10) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_half* const w = r.half_or_null(a[1]);
  const int H = r.integer(a[2]);
  const Table X = r.table(a[3]), Y = r.table(a[4]);
  const auto op = hgnn_reduce(r.integer(a[5]));
  const float* const scale = r.single_or_null(a[6]);
  const int F = r.integer_or(a[7], X.cols);
  size_t bytes = 0;
  void* const ws = a[8] == Py_None ? nullptr : r.workspace(a[8], &bytes);
  void* const s = r.stream(a[9]);
  return [=] { return f_spmm(&g, w, H, X.half(), X.ld, Y.half(), Y.ld, F, op, scale, ws, bytes, s); };
} HGNN_END

HGNN_CALL(spmm_discretized, 10) {
  const hgnn_plan* const p = r.plan(a[0]);
  const hgnn_csr g = r.graph(a[1]);
  const hgnn_half* const w = r.half_or_null(a[2]);
  const int H = r.integer(a[3]);
  const Table X = r.table(a[4]), Y = r.table(a[5]);
  const auto op = hgnn_reduce(r.integer(a[6]));
  const float* const scale = r.single_or_null(a[7]);
  const int F = r.integer_or(a[8], X.cols);
  void* const s = r.stream(a[9]);
  return [=] { return f_spmm_discretized(p, &g, w, H, X.half(), X.ld, Y.half(), Y.ld, F, op, scale, s); };
} HGNN_END

HGNN_CALL(spmm_discretized_fused, 15) {
  const hgnn_plan* const p = r.plan(a[0]);
  const hgnn_csr g = r.graph(a[1]);
  const hgnn_half* const w = r.half_or_null(a[2]);
  const int H = r.integer(a[3]);
  const Table X = r.table(a[4]), Y = r.table(a[5]);
  const auto op = hgnn_reduce(r.integer(a[6]));
  const float* const scale = r.single_or_null(a[7]);
  const float* const col_scale = r.single_or_null(a[8]);
  const Table self = r.table_or_null(a[9]);
  const float self_coef = r.real(a[10]), agg_coef = r.real(a[11]);
  const int F = r.integer_or(a[12], X.cols);
  const Table scaled = r.table_or_null(a[13]);
  void* const s = r.stream(a[14]);
  const hgnn_spmm_fusion fz{col_scale, self.half(), self.ld, self_coef, agg_coef, scaled.half(), scaled.ld};
  return [=] { return f_spmm_discretized_fused(p, &g, w, H, X.half(), X.ld, Y.half(), Y.ld, F, op, scale, &fz, s); };
} HGNN_END

HGNN_CALL(sddmm, 12) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan_or_null(a[1]);
  const auto op = hgnn_sddmm_op(r.integer(a[2]));
  const int H = r.integer(a[3]), D = r.integer(a[4]);
  const Table U = r.table(a[5]), V = r.table(a[6]);
  hgnn_half* const out = r.half(a[7]);
  const hgnn_half *const al = r.half_or_null(a[8]), *const ar = r.half_or_null(a[9]);
  const float slope = r.real(a[10]);
  void* const s = r.stream(a[11]);
  return [=] { return f_sddmm(&g, p, op, H, D, U.half(), U.ld, V.half(), V.ld, al, ar, slope, out, s); };
} HGNN_END

HGNN_CALL(edge_softmax, 6) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan_or_null(a[1]);
  const int H = r.integer(a[2]);
  hgnn_half *const e = r.half(a[3]), *const alpha = r.half(a[4]);
  void* const s = r.stream(a[5]);
  return [=] { return f_edge_softmax(&g, p, H, e, alpha, s); };
} HGNN_END

HGNN_CALL(edge_softmax_bwd, 9) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan_or_null(a[1]);
  const int H = r.integer(a[2]);
  hgnn_half *const alpha = r.half(a[3]), *const dalpha = r.half(a[4]), *const de = r.half(a[5]), *const e = r.half_or_null(a[6]);
  const float slope = r.real(a[7]);
  void* const s = r.stream(a[8]);
  return [=] { return f_edge_softmax_bwd(&g, p, H, alpha, dalpha, e, slope, de, s); };
} HGNN_END

HGNN_CALL(edge_rowsum, 6) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan_or_null(a[1]);
  const int H = r.integer(a[2]);
  hgnn_half *const t = r.half(a[3]), *const out = r.half(a[4]);
  void* const s = r.stream(a[5]);
  return [=] { return f_edge_rowsum(&g, p, H, t, out, s); };
} HGNN_END

HGNN_CALL(edge_colsum, 6) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan(a[1]);
  const int H = r.integer(a[2]);
  hgnn_half *const t = r.half(a[3]), *const out = r.half(a[4]);
  void* const s = r.stream(a[5]);
  return [=] { return f_edge_colsum(&g, p, H, t, out, s); };
} HGNN_END

HGNN_CALL(gat_forward_fused, 12) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan(a[1]);
  const int H = r.integer(a[2]), D = r.integer(a[3]);
  const Table U = r.table(a[4]), V = r.table(a[5]);
  const hgnn_half *const al = r.half(a[6]), *const ar = r.half(a[7]);
  const Table out = r.table(a[8]);
  float* const lse = r.single_or_null(a[9]);
  const float slope = r.real(a[10]);
  void* const s = r.stream(a[11]);
  return [=] { return f_gat_forward_fused(&g, p, H, D, U.half(), U.ld, V.half(), V.ld, al, ar, slope, out.half(), out.ld, lse, s); };
} HGNN_END

HGNN_CALL(gat_forward_fused_save, 14) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan(a[1]);
  const int H = r.integer(a[2]), D = r.integer(a[3]);
  const Table U = r.table(a[4]), V = r.table(a[5]);
  const hgnn_half *const al = r.half(a[6]), *const ar = r.half(a[7]);
  const Table out = r.table(a[8]);
  float* const lse = r.single(a[9]);
  const Table masked = r.table(a[10]);
  float* const csum = r.single(a[11]);
  const float slope = r.real(a[12]);
  void* const s = r.stream(a[13]);
  return [=] {
    return f_gat_forward_fused_save(&g, p, H, D, U.half(), U.ld, V.half(), V.ld, al, ar, slope, out.half(), out.ld, lse, masked.half(), masked.ld, csum, s);
  };
} HGNN_END

HGNN_CALL(gat_backward_fused_saved, 20) {
  const hgnn_csr g = r.graph(a[0]);
  const hgnn_plan* const p = r.plan(a[1]);
  const hgnn_csr gt = r.graph(a[2]);
  const hgnn_plan* const pt = r.plan(a[3]);
  const int H = r.integer(a[4]), D = r.integer(a[5]);
  const Table U = r.table(a[6]), V = r.table(a[7]);
  const hgnn_half *const al = r.half(a[8]), *const ar = r.half(a[9]);
  const Table out = r.table(a[10]);
  const float* const lse = r.single(a[11]);
  const Table masked = r.table(a[12]);
  const float* const csum = r.single(a[13]);
  const Table dOut = r.table(a[14]), dV = r.table(a[15]);
  hgnn_half *const d_el = r.half(a[16]), *const d_er = r.half(a[17]);
  const float slope = r.real(a[18]);
  void* const s = r.stream(a[19]);
  return [=] {
    return f_gat_backward_fused_saved(&g, p, &gt, pt, H, D, U.half(), U.ld, V.half(), V.ld, al, ar, slope, out.half(), out.ld, lse, masked.half(),
                                      masked.ld, csum, dOut.half(), dOut.ld, dV.half(), dV.ld, d_el, d_er, s);
  };
} HGNN_END

HGNN_CALL(gat_feature_grad, 13) {
  const int H = r.integer(a[0]), D = r.integer(a[1]);
  const Table dV = r.table(a[2]);
  const hgnn_half *const d_el = r.half(a[3]), *const d_er = r.half(a[4]), *const al = r.half(a[5]), *const ar = r.half(a[6]);
  const Table h = r.table(a[7]), dh = r.table(a[8]);
  float *const da_l = r.single(a[9]), *const da_r = r.single(a[10]);
  size_t bytes;
  void* const ws = r.workspace(a[11], &bytes);
  void* const s = r.stream(a[12]);
  return [=] { return f_gat_feature_grad(dV.rows, H, D, dV.half(), dV.ld, d_el, d_er, al, ar, h.half(), h.ld, dh.half(), dh.ld, da_l, da_r, ws, bytes, s); };
} HGNN_END

// bind({entry point: address}, raw stream of a device, current device)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3 || !PyDict_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "bind(dict, callable, callable)");
    return nullptr;
  }
#define HGNN_BIND(name)                                                                 \
  {                                                                                     \
    PyObject* const v = PyDict_GetItemString(a[0], "hgnn_" #name);                      \
    void* const p = v && PyLong_Check(v) ? PyLong_AsVoidPtr(v) : nullptr;               \
    if (!p) {                                                                           \
      PyErr_SetString(PyExc_KeyError, "hgnn_" #name);                                   \
      return nullptr;                                                                   \
    }                                                                                   \
    f_##name = reinterpret_cast<decltype(f_##name)>(p);                                 \
  }
  HGNN_ENTRIES(HGNN_BIND)
  g_current_device = Py_NewRef(a[2]);
  g_raw_stream = Py_NewRef(a[1]);
  Py_RETURN_NONE;
}

#define HGNN_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HGNN_METHOD(bind), HGNN_METHOD(linear), HGNN_METHOD(linear_wgrad), HGNN_METHOD(spmm), HGNN_METHOD(spmm_discretized),
                         HGNN_METHOD(spmm_discretized_fused), HGNN_METHOD(sddmm), HGNN_METHOD(edge_softmax), HGNN_METHOD(edge_softmax_bwd),
                         HGNN_METHOD(edge_rowsum), HGNN_METHOD(edge_colsum), HGNN_METHOD(gat_forward_fused), HGNN_METHOD(gat_forward_fused_save),
                         HGNN_METHOD(gat_backward_fused_saved), HGNN_METHOD(gat_feature_grad), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  g_struct = PyUnicode_InternFromString("struct");
  g_handle = PyUnicode_InternFromString("handle");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return PyModule_Create(&module);
}
