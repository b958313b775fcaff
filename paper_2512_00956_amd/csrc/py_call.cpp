// The per-step entry points of wush.h as Python functions: pointers, sizes and strides are read off the tensors here
// instead of one Python attribute at a time.  A layer call of a small batch takes the GPU 6 us, and marshalling its 15
// arguments through ctypes took the host 5 to 6 of its 12 (now about 1.5).  Marshalling only: every function passes its
// arguments on and returns the status code; binding.py raises.
//
// Tensors are torch tensors (anything with data_ptr(), shape, stride(), numel(), element_size()); None is a null pointer.
// A format descriptor is binding.WushFmt (by its bytes) or None for the default.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/wush.h"

namespace {

PyObject *s_data_ptr, *s_shape, *s_stride, *s_numel, *s_element_size, *o_zero;
PyObject* format_type;   // binding.WushFmt, set when binding loads this module

// Conversions: false with an exception set on failure.
bool to_i64(PyObject* o, int64_t* out) {
  *out = PyLong_AsLongLong(o);
  return !(*out == -1 && PyErr_Occurred());
}
bool call_i64(PyObject* t, PyObject* method, int64_t* out) {
  PyObject* args[1] = {t};
  PyObject* r = PyObject_VectorcallMethod(method, args, 1, nullptr);
  if (!r) return false;
  const bool ok = to_i64(r, out);
  Py_DECREF(r);
  return ok;
}
template <class T>
bool ptr(PyObject* t, T** out) {
  if (t == Py_None) {
    *out = nullptr;
    return true;
  }
  PyObject* args[1] = {t};
  PyObject* r = PyObject_VectorcallMethod(s_data_ptr, args, 1, nullptr);
  if (!r) return false;
  *out = static_cast<T*>(PyLong_AsVoidPtr(r));
  Py_DECREF(r);
  return !PyErr_Occurred();
}
bool shape2(PyObject* t, int64_t* rows, int64_t* cols) {
  PyObject* s = PyObject_GetAttr(t, s_shape);
  if (!s) return false;
  bool ok = PyTuple_Check(s) && PyTuple_GET_SIZE(s) == 2;
  if (!ok) PyErr_SetString(PyExc_ValueError, "a two-dimensional tensor is expected");
  ok = ok && to_i64(PyTuple_GET_ITEM(s, 0), rows) && to_i64(PyTuple_GET_ITEM(s, 1), cols);
  Py_DECREF(s);
  return ok;
}
bool row_stride(PyObject* t, int64_t* out) {
  PyObject* args[2] = {t, o_zero};
  PyObject* r = PyObject_VectorcallMethod(s_stride, args, 2, nullptr);
  if (!r) return false;
  const bool ok = to_i64(r, out);
  Py_DECREF(r);
  return ok;
}
// size of the second dimension
bool columns(PyObject* t, int64_t* out) {
  PyObject* s = PyObject_GetAttr(t, s_shape);
  if (!s) return false;
  bool ok = PyTuple_Check(s) && PyTuple_GET_SIZE(s) >= 2;
  if (!ok) PyErr_SetString(PyExc_IndexError, "a tensor of at least two dimensions is expected");
  ok = ok && to_i64(PyTuple_GET_ITEM(s, 1), out);
  Py_DECREF(s);
  return ok;
}
// K as given, or from the canonical shape of the packed codes
bool k_of(PyObject* k, PyObject* codes, int64_t* out) {
  if (k != Py_None) return to_i64(k, out);
  PyObject* s = PyObject_GetAttr(codes, s_shape);
  if (!s) return false;
  bool ok = PyTuple_Check(s) && PyTuple_GET_SIZE(s) > 0;
  if (!ok) PyErr_SetString(PyExc_IndexError, "codes without a shape");
  ok = ok && to_i64(PyTuple_GET_ITEM(s, PyTuple_GET_SIZE(s) - 1), out);
  if (ok) *out *= 2;
  Py_DECREF(s);
  return ok;
}
bool nbytes(PyObject* t, size_t* out) {
  int64_t n = 0, e = 0;
  if (t != Py_None && !(call_i64(t, s_numel, &n) && call_i64(t, s_element_size, &e))) return false;
  *out = static_cast<size_t>(n * e);
  return true;
}
bool format(PyObject* f, int32_t default_layout, wush_fmt* out) {
  if (f == Py_None) {
    *out = wush_default_fmt();
    out->layout = default_layout;
    return true;
  }
  Py_buffer b;
  const int type = format_type ? PyObject_IsInstance(f, format_type) : 0;
  if (type < 0) return false;
  if (!type) {
    PyErr_SetString(PyExc_TypeError, "a WushFmt is expected");
    return false;
  }
  if (PyObject_GetBuffer(f, &b, PyBUF_SIMPLE) != 0) return false;
  const bool ok = b.len >= static_cast<Py_ssize_t>(sizeof(wush_fmt));
  if (ok) *out = *static_cast<const wush_fmt*>(b.buf);
  else PyErr_SetString(PyExc_TypeError, "a WushFmt is expected");
  PyBuffer_Release(&b);
  return ok;
}
bool arity(const char* name, Py_ssize_t got, Py_ssize_t want) {
  if (got == want) return true;
  PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, want, got);
  return false;
}
bool to_i32(PyObject* o, int32_t* out) {
  int64_t v;
  if (!to_i64(o, &v)) return false;
  *out = static_cast<int32_t>(v);
  return true;
}

#define WUSH_CALL(expr)     \
  wush_status st;           \
  Py_BEGIN_ALLOW_THREADS    \
  st = (expr);              \
  Py_END_ALLOW_THREADS      \
  return PyLong_FromLong(st)

// (X, T_blocks, Xq, Xs, fmt, dbg_Yt, stream)
PyObject* quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, K, ld;
  void *X, *T, *Xq, *Xs;
  float* dbg;
  wush_fmt f;
  if (!arity("quantize_act", n, 7) || !shape2(a[0], &M, &K) || !row_stride(a[0], &ld) || !ptr(a[0], &X) || !ptr(a[1], &T) ||
      !ptr(a[2], &Xq) || !ptr(a[3], &Xs) || !format(a[4], WUSH_LAYOUT_CANONICAL, &f) || !ptr(a[5], &dbg))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[6]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_quantize_act(X, M, K, ld, T, f, Xq, Xs, dbg, stream));
}

// (Xq, Xs, Wq, Ws, Y, fmt, stream, K)
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, N, K, ld;
  void *Xq, *Xs, *Wq, *Ws, *Y;
  wush_fmt f;
  if (!arity("linear", n, 8) || !shape2(a[4], &M, &N) || !row_stride(a[4], &ld) || !k_of(a[7], a[0], &K) || !ptr(a[0], &Xq) ||
      !ptr(a[1], &Xs) || !ptr(a[2], &Wq) || !ptr(a[3], &Ws) || !ptr(a[4], &Y) || !format(a[5], WUSH_LAYOUT_CANONICAL, &f))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[6]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_linear(Xq, Xs, Wq, Ws, M, N, K, f, Y, ld, stream));
}

// (X, T_blocks, Wq, Ws, Y, workspace, fmt, stream)
PyObject* layer_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, K, ldx, N, ldy;
  void *X, *T, *Wq, *Ws, *Y, *w;
  size_t bytes;
  wush_fmt f;
  if (!arity("layer_decode", n, 8) || !shape2(a[0], &M, &K) || !row_stride(a[0], &ldx) || !columns(a[4], &N) ||
      !row_stride(a[4], &ldy) || !ptr(a[0], &X) || !ptr(a[1], &T) || !ptr(a[2], &Wq) || !ptr(a[3], &Ws) || !ptr(a[4], &Y) ||
      !ptr(a[5], &w) || !nbytes(a[5], &bytes) || !format(a[6], WUSH_LAYOUT_TILED, &f))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[7]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_layer_decode(X, M, K, ldx, T, Wq, Ws, N, f, Y, ldy, w, bytes, stream));
}

// (X, T_blocks, Wq, Ws, Y, fmt, stream)
PyObject* layer_decode_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, K, ldx, N, ldy;
  void *X, *T, *Wq, *Ws, *Y;
  wush_fmt f;
  if (!arity("layer_decode_static", n, 7) || !shape2(a[0], &M, &K) || !row_stride(a[0], &ldx) || !columns(a[4], &N) ||
      !row_stride(a[4], &ldy) || !ptr(a[0], &X) || !ptr(a[1], &T) || !ptr(a[2], &Wq) || !ptr(a[3], &Ws) || !ptr(a[4], &Y) ||
      !format(a[5], WUSH_LAYOUT_TILED, &f))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[6]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_layer_decode_static(X, M, K, ldx, T, Wq, Ws, N, f, Y, ldy, stream));
}

// (X, T16, tensor_scale, Xq, Xs, layout, dbg_Yt, stream)
PyObject* quantize_act_nvfp4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, K, ld;
  void *X, *T, *Xq, *Xs;
  float *ts, *dbg;
  int32_t layout;
  if (!arity("quantize_act_nvfp4", n, 8) || !shape2(a[0], &M, &K) || !row_stride(a[0], &ld) || !ptr(a[0], &X) || !ptr(a[1], &T) ||
      !ptr(a[2], &ts) || !ptr(a[3], &Xq) || !ptr(a[4], &Xs) || !to_i32(a[5], &layout) || !ptr(a[6], &dbg))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[7]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_quantize_act_nvfp4(X, M, K, ld, T, ts, layout, Xq, Xs, dbg, stream));
}

// (Xq, Xs, tsx, Wq, Ws, tsw, Y, layout, out_dtype, stream, K)
PyObject* linear_nvfp4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, N, K, ld;
  void *Xq, *Xs, *Wq, *Ws, *Y;
  float *tsx, *tsw;
  int32_t layout, out;
  if (!arity("linear_nvfp4", n, 11) || !shape2(a[6], &M, &N) || !row_stride(a[6], &ld) || !k_of(a[10], a[0], &K) ||
      !ptr(a[0], &Xq) || !ptr(a[1], &Xs) || !ptr(a[2], &tsx) || !ptr(a[3], &Wq) || !ptr(a[4], &Ws) || !ptr(a[5], &tsw) ||
      !ptr(a[6], &Y) || !to_i32(a[7], &layout) || !to_i32(a[8], &out))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[9]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_linear_nvfp4(Xq, Xs, tsx, Wq, Ws, tsw, M, N, K, layout, out, Y, ld, stream));
}

// (X, T_blocks, Xq, Xs, layout, dbg_Yt, stream)
PyObject* quantize_act_int4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, K, ld;
  void *X, *T, *Xq, *Xs;
  float* dbg;
  int32_t layout;
  if (!arity("quantize_act_int4", n, 7) || !shape2(a[0], &M, &K) || !row_stride(a[0], &ld) || !ptr(a[0], &X) || !ptr(a[1], &T) ||
      !ptr(a[2], &Xq) || !ptr(a[3], &Xs) || !to_i32(a[4], &layout) || !ptr(a[5], &dbg))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[6]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_quantize_act_int4(X, M, K, ld, T, layout, Xq, Xs, dbg, stream));
}

// (Xq, Xs, Wq, Ws, Y, layout, out_dtype, stream, K)
PyObject* linear_int4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t M, N, K, ld;
  void *Xq, *Xs, *Wq, *Ws, *Y;
  int32_t layout, out;
  if (!arity("linear_int4", n, 9) || !shape2(a[4], &M, &N) || !row_stride(a[4], &ld) || !k_of(a[8], a[0], &K) || !ptr(a[0], &Xq) ||
      !ptr(a[1], &Xs) || !ptr(a[2], &Wq) || !ptr(a[3], &Ws) || !ptr(a[4], &Y) || !to_i32(a[5], &layout) || !to_i32(a[6], &out))
    return nullptr;
  void* stream = PyLong_AsVoidPtr(a[7]);
  if (PyErr_Occurred()) return nullptr;
  WUSH_CALL(wush_linear_int4(Xq, Xs, Wq, Ws, M, N, K, layout, out, Y, ld, stream));
}

// (type): the class format descriptors are instances of
PyObject* use_format_type(PyObject*, PyObject* type) {
  Py_INCREF(type);
  Py_XSETREF(format_type, type);
  Py_RETURN_NONE;
}

#define WUSH_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {WUSH_METHOD(quantize_act),       WUSH_METHOD(linear),       WUSH_METHOD(layer_decode),
                         WUSH_METHOD(layer_decode_static), WUSH_METHOD(quantize_act_nvfp4), WUSH_METHOD(linear_nvfp4),
                         WUSH_METHOD(quantize_act_int4),  WUSH_METHOD(linear_int4),
                         {"use_format_type", use_format_type, METH_O, nullptr},            {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_wush_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__wush_call(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_shape = PyUnicode_InternFromString("shape");
  s_stride = PyUnicode_InternFromString("stride");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  o_zero = PyLong_FromLong(0);
  if (!s_data_ptr || !s_shape || !s_stride || !s_numel || !s_element_size || !o_zero) return nullptr;
  return PyModule_Create(&module);
}
