// The calls a generated token is made of, marshalled natively for Python: a call of hi_decode_group that the library refuses at once
// takes 2.5 us through ctypes and the checks around it, 0.63 this way (1.25 and 0.30 on a faster host); a layer of a short decode
// takes 13.  Arguments are the usual ones - ints, None, tensors (their
// data_ptr), streams (their cuda_stream), the context as ctypes.c_void_p; for anything else a call returns None without
// calling anything, and the caller goes through ctypes, which accepts, refuses and reports as it always did.  The library's
// functions are given as addresses (bind), and the interpreter lock is released while they run, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cstdint>
#include "headinfer.h"

namespace {

decltype(&hi_prefill_group) f_prefill;
decltype(&hi_decode_group) f_decode;
decltype(&hi_decode_group_ragged) f_ragged;
decltype(&hi_qkv_rope) f_qkv;
decltype(&hi_out_proj) f_out;
PyObject *s_data_ptr, *s_cuda_stream, *s_value, *c_void_p_type;

// One call's arguments.  ok goes down at the first unusual one; a Python error (of a data_ptr, say) is kept and raised.
struct Args {
  PyObject* const* a;
  bool ok = true;
  int64_t integer(Py_ssize_t i) {
    if (!ok || !PyLong_Check(a[i])) { ok = false; return 0; }
    const long long v = PyLong_AsLongLong(a[i]);
    if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
    return v;
  }
  int32_t int32(Py_ssize_t i) {
    const int64_t v = integer(i);
    if (v != (int32_t)v) ok = false;
    return (int32_t)v;
  }
  double real(Py_ssize_t i) {
    if (!ok || !PyFloat_CheckExact(a[i])) { ok = false; return 0; }
    return PyFloat_AS_DOUBLE(a[i]);
  }
  void* address(PyObject* x) {
    if (x == Py_None) return nullptr;
    void* const p = PyLong_Check(x) ? PyLong_AsVoidPtr(x) : nullptr;
    if (!PyLong_Check(x) || (!p && PyErr_Occurred())) { PyErr_Clear(); ok = false; }
    return p;
  }
  void* from(PyObject* got) {                     // a new reference or an error
    if (!got) { ok = false; return nullptr; }
    void* const p = address(got);
    Py_DECREF(got);
    return p;
  }
  void* buffer(Py_ssize_t i) {
    if (!ok || a[i] == Py_None || PyLong_Check(a[i])) return ok ? address(a[i]) : nullptr;
    return from(PyObject_CallMethodNoArgs(a[i], s_data_ptr));
  }
  void* stream(Py_ssize_t i) {
    if (!ok || a[i] == Py_None || PyLong_Check(a[i])) return ok ? address(a[i]) : nullptr;
    return from(PyObject_GetAttr(a[i], s_cuda_stream));
  }
  hi_ctx* context(Py_ssize_t i) {
    if (!ok || a[i] == Py_None || PyLong_Check(a[i])) return ok ? (hi_ctx*)address(a[i]) : nullptr;
    if ((PyObject*)Py_TYPE(a[i]) != c_void_p_type) { ok = false; return nullptr; }
    return (hi_ctx*)from(PyObject_GetAttr(a[i], s_value));
  }
};

template <class F>
PyObject* run(const Args& g, F&& call) {
  if (PyErr_Occurred()) return nullptr;
  if (!g.ok) Py_RETURN_NONE;
  hi_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

PyObject* prefill_group(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!f_prefill || n != 14) Py_RETURN_NONE;
  Args g{a};
  hi_ctx* c = g.context(0);
  const int32_t layer = g.int32(1), head = g.int32(2), nh = g.int32(3);
  void *q = g.buffer(4), *k = g.buffer(5), *v = g.buffer(6);
  const int64_t past = g.integer(7);
  const int32_t len = g.int32(8);
  void* out = g.buffer(9);
  const int32_t nl = g.int32(10), nhead = g.int32(11), nn = g.int32(12);
  const int64_t npast = g.integer(13);
  return run(g, [&] { return f_prefill(c, layer, head, nh, q, k, v, past, len, out, nl, nhead, nn, npast); });
}

PyObject* decode_group(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!f_decode || n != 13) Py_RETURN_NONE;
  Args g{a};
  hi_ctx* c = g.context(0);
  const int32_t layer = g.int32(1), head = g.int32(2), nh = g.int32(3);
  void *q = g.buffer(4), *k = g.buffer(5), *v = g.buffer(6);
  const int64_t past = g.integer(7);
  void* out = g.buffer(8);
  const int32_t nl = g.int32(9), nhead = g.int32(10), nn = g.int32(11);
  const int64_t npast = g.integer(12);
  return run(g, [&] { return f_decode(c, layer, head, nh, q, k, v, past, out, nl, nhead, nn, npast); });
}

PyObject* decode_group_ragged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!f_ragged || n != 9) Py_RETURN_NONE;
  Args g{a};
  hi_ctx* c = g.context(0);
  const int32_t layer = g.int32(1), head = g.int32(2), nh = g.int32(3);
  void *q = g.buffer(4), *k = g.buffer(5), *v = g.buffer(6), *out = g.buffer(8);
  constexpr int kMost = 256;                     // (the library takes 64)
  int64_t lens[kMost];
  if (g.ok && PyList_CheckExact(a[7]) && PyList_GET_SIZE(a[7]) == nh && nh >= 1 && nh <= kMost) {
    for (int j = 0; j < nh; ++j) {
      Args one{&PyList_GET_ITEM(a[7], j)};
      lens[j] = one.integer(0);
      g.ok = g.ok && one.ok;
    }
  } else {
    g.ok = false;
  }
  return run(g, [&] { return f_ragged(c, layer, head, nh, q, k, v, lens, out); });
}

PyObject* qkv_rope(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!f_qkv || n != 15) Py_RETURN_NONE;
  Args g{a};
  void *s = g.stream(0), *x = g.buffer(1), *w = g.buffer(2);
  const int32_t d = g.int32(3), hq = g.int32(4), hkv = g.int32(5), len = g.int32(6);
  const int64_t past = g.integer(7);
  const double theta = g.real(8);
  const int32_t fp32 = g.int32(9);
  void *q = g.buffer(10), *k = g.buffer(11), *v = g.buffer(12), *ws = g.buffer(13);
  const float scale = (float)g.real(14);
  return run(g, [&] { return f_qkv(s, x, w, d, hq, hkv, len, past, theta, fp32, q, k, v, ws, scale); });
}

PyObject* out_proj(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!f_out || n != 8) Py_RETURN_NONE;
  Args g{a};
  void *s = g.stream(0), *x = g.buffer(1), *w = g.buffer(2);
  const int32_t hq = g.int32(3), d = g.int32(4), len = g.int32(5), fp32 = g.int32(6);
  void* y = g.buffer(7);
  return run(g, [&] { return f_out(s, x, w, hq, d, len, fp32, y); });
}

// bind(prefill_group, decode_group, decode_group_ragged, qkv_rope, out_proj, ctypes.c_void_p): the functions' addresses
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 6) { PyErr_SetString(PyExc_TypeError, "bind takes five addresses and a type"); return nullptr; }
  void* p[5];
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address"); return nullptr; }
  }
  f_prefill = (decltype(f_prefill))p[0];
  f_decode = (decltype(f_decode))p[1];
  f_ragged = (decltype(f_ragged))p[2];
  f_qkv = (decltype(f_qkv))p[3];
  f_out = (decltype(f_out))p[4];
  Py_INCREF(a[5]);
  Py_XSETREF(c_void_p_type, a[5]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"prefill_group", (PyCFunction)(void (*)(void))prefill_group, METH_FASTCALL, nullptr},
    {"decode_group", (PyCFunction)(void (*)(void))decode_group, METH_FASTCALL, nullptr},
    {"decode_group_ragged", (PyCFunction)(void (*)(void))decode_group_ragged, METH_FASTCALL, nullptr},
    {"qkv_rope", (PyCFunction)(void (*)(void))qkv_rope, METH_FASTCALL, nullptr},
    {"out_proj", (PyCFunction)(void (*)(void))out_proj, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_value = PyUnicode_InternFromString("value");
  if (!s_data_ptr || !s_cuda_stream || !s_value) return nullptr;
  return PyModule_Create(&module_def);
}
