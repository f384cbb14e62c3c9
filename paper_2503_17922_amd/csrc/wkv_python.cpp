// CPython entry to the calls a program makes per layer or per token (module `_native` of the package).
// Marshalling only: tensors become raw device pointers, sequences of tensors arrays on the stack, and the
// call goes to the C ABI with the interpreter lock released.  A decode step enqueues two kernels in 5 us of host
// time; converting its thirteen arguments through ctypes and asking torch for the stream took another 4.5 us,
// here both take about 1 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>

#include "wkv.h"

namespace {

PyObject *s_c, *s_data_ptr, *s_numel, *s_element_size;        // interned attribute names
PyObject *slow_stream;                                        // callable: the current stream by torch's public API
PyObject *get_device, *get_raw_stream;                        // torch._C functions behind it, once torch has initialised the GPU
PyObject *convert;                                            // callable (o, structure type): what ctypes takes from o.ref()

// Every converter returns false with a Python exception set.
// The structure behind a Problem or DecodeShape, held until the call is over.  Taken from `.c` as it is now (an object
// may be copied or given another structure), of exactly this type; anything else goes to `convert`, which accepts and
// refuses what a ctypes call of the same function does.
struct Kind { PyObject *wrapper, *structure; };
Kind problem_kind, shape_kind;
struct Structure {
  Py_buffer view;
  Structure() { view.obj = nullptr; }
  ~Structure() { if (view.obj) PyBuffer_Release(&view); }
  Structure(const Structure &) = delete;
  bool fill(PyObject *o, const Kind &kind) {
    PyObject *c = nullptr;
    if ((PyObject *)Py_TYPE(o) == kind.wrapper && !(c = PyObject_GetAttr(o, s_c))) return false;
    if (!c || (PyObject *)Py_TYPE(c) != kind.structure) {
      Py_XDECREF(c);
      if (!convert) { PyErr_SetString(PyExc_RuntimeError, "bind was not called"); return false; }
      if (!(c = PyObject_CallFunctionObjArgs(convert, o, kind.structure, nullptr))) return false;
    }
    const bool ok = PyObject_GetBuffer(c, &view, PyBUF_SIMPLE) == 0;
    Py_DECREF(c);                                // the buffer keeps it
    return ok;
  }
  const wkv_problem *problem() const { return (const wkv_problem *)view.buf; }
  const wkv_decode_shape *shape() const { return (const wkv_decode_shape *)view.buf; }
};

bool pointer(PyObject *o, void **out) {
  if (o == Py_None) { *out = nullptr; return true; }
  PyObject *v = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!v) return false;
  *out = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

bool call_size(PyObject *o, PyObject *name, size_t *out) {
  PyObject *v = PyObject_CallMethodNoArgs(o, name);
  if (!v) return false;
  *out = PyLong_AsSize_t(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

bool workspace(PyObject *o, void **out, size_t *bytes) {
  *bytes = 0;
  if (!pointer(o, out)) return false;
  size_t n = 0, e = 0;
  if (o != Py_None) {
    if (!call_size(o, s_numel, &n) || !call_size(o, s_element_size, &e)) return false;
    *bytes = n * e;
  }
  return true;
}

bool integer(PyObject *o, int32_t *out) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) return false;
  if (v < INT32_MIN || v > INT32_MAX) { PyErr_SetString(PyExc_OverflowError, "integer out of range"); return false; }
  *out = (int32_t)v;
  return true;
}

// A sequence of at most CAP tensors (or None); a library call that asks for more than it holds finds NULL there.
template <int CAP>
struct Pointers {
  void *p[CAP];
  Py_ssize_t n = 0;
  bool fill(PyObject *seq) {
    std::memset(p, 0, sizeof p);
    PyObject *f = PySequence_Fast(seq, "expected a sequence of tensors");
    if (!f) return false;
    n = PySequence_Fast_GET_SIZE(f);
    bool ok = true;
    for (Py_ssize_t i = 0; ok && i < n && i < CAP; ++i) ok = pointer(PySequence_Fast_GET_ITEM(f, i), &p[i]);
    Py_DECREF(f);
    return ok;
  }
};

bool stream_of(PyObject *o, void **out) {
  if (o != Py_None) {
    PyObject *i = PyNumber_Long(o);
    if (!i) return false;
    *out = PyLong_AsVoidPtr(i);
    Py_DECREF(i);
    return !PyErr_Occurred();
  }
  PyObject *v;
  if (get_raw_stream) {
    PyObject *dev = PyObject_CallNoArgs(get_device);
    if (!dev) return false;
    v = PyObject_CallOneArg(get_raw_stream, dev);
    Py_DECREF(dev);
  } else {
    if (!slow_stream) { PyErr_SetString(PyExc_RuntimeError, "bind was not called"); return false; }
    v = PyObject_CallNoArgs(slow_stream);        // initialises torch's GPU side where that has not happened yet
  }
  if (!v) return false;
  *out = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  if (PyErr_Occurred()) return false;
  if (!get_raw_stream) {
    PyObject *m = PyImport_ImportModule("torch._C");
    PyObject *d = m ? PyObject_GetAttrString(m, "_cuda_getDevice") : nullptr;
    PyObject *r = d ? PyObject_GetAttrString(m, "_cuda_getCurrentRawStream") : nullptr;
    Py_XDECREF(m);
    if (r) { get_device = d; get_raw_stream = r; }
    else { Py_XDECREF(d); PyErr_Clear(); }       // a torch without them: the public API every time
  }
  return true;
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return false;
}

template <class F>
PyObject *call(F &&f) {
  wkv_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// (shape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, workspace, stream)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure sh;
  void *t[7], *ws, *st;
  size_t bytes;
  if (!arity(n, 10) || !sh.fill(a[0], shape_kind)) return nullptr;
  for (int i = 0; i < 7; ++i) if (!pointer(a[1 + i], &t[i])) return nullptr;
  if (!workspace(a[8], &ws, &bytes) || !stream_of(a[9], &st)) return nullptr;
  return call([&] { return wkv_decode_step(sh.shape(), t[0], t[1], t[2], t[3], t[4], (int32_t *)t[5], (float *)t[6], ws, bytes, st); });
}

// (shape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, stream)
PyObject *decode_step_static(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure sh;
  void *t[7], *st;
  if (!arity(n, 9) || !sh.fill(a[0], shape_kind)) return nullptr;
  for (int i = 0; i < 7; ++i) if (!pointer(a[1 + i], &t[i])) return nullptr;
  if (!stream_of(a[8], &st)) return nullptr;
  return call([&] { return wkv_decode_step_static(sh.shape(), t[0], t[1], t[2], t[3], t[4], (int32_t *)t[5], (float *)t[6], st); });
}

// (problem, q_obs, k_first, lse_obs, t_out, workspace, stream)
PyObject *score(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *t[4], *ws, *st;
  size_t bytes;
  if (!arity(n, 7) || !pr.fill(a[0], problem_kind)) return nullptr;
  for (int i = 0; i < 4; ++i) if (!pointer(a[1 + i], &t[i])) return nullptr;
  if (!workspace(a[5], &ws, &bytes) || !stream_of(a[6], &st)) return nullptr;
  return call([&] { return wkv_score(pr.problem(), t[0], t[1], (const float *)t[2], (float *)t[3], ws, bytes, st); });
}

// (problem, t, s_out, stream)
PyObject *window_pool(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *t, *s, *st;
  if (!arity(n, 4) || !pr.fill(a[0], problem_kind) || !pointer(a[1], &t) || !pointer(a[2], &s) || !stream_of(a[3], &st)) return nullptr;
  return call([&] { return wkv_window_pool(pr.problem(), (const float *)t, (float *)s, st); });
}

// (problem, s, win_idx_out, tok_idx_out, n_keep_out, stream)
PyObject *topk_windows(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *t[4], *st;
  if (!arity(n, 6) || !pr.fill(a[0], problem_kind)) return nullptr;
  for (int i = 0; i < 4; ++i) if (!pointer(a[1 + i], &t[i])) return nullptr;
  if (!stream_of(a[5], &st)) return nullptr;
  return call([&] { return wkv_topk_windows(pr.problem(), (const float *)t[0], (int32_t *)t[1], (int32_t *)t[2], (int32_t *)t[3], st); });
}

// (problem, k_layers, v_layers, tok_idx, n_keep, k_out_layers, v_out_layers, stream)
PyObject *gather_group(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *ti, *nk, *st;
  Pointers<WKV_MAX_LAYERS> k, v, ko, vo;
  if (!arity(n, 8) || !pr.fill(a[0], problem_kind) || !k.fill(a[1]) || !v.fill(a[2]) || !pointer(a[3], &ti) || !pointer(a[4], &nk) ||
      !ko.fill(a[5]) || !vo.fill(a[6]) || !stream_of(a[7], &st)) return nullptr;
  const int32_t layers = (int32_t)(k.n > WKV_MAX_LAYERS ? WKV_MAX_LAYERS + 1 : k.n);
  return call([&] { return wkv_gather_group(pr.problem(), layers, k.p, v.p, (const int32_t *)ti, (const int32_t *)nk, ko.p, vo.p, st); });
}

// (problem, gamma, q_obs, lse_obs, k_layers, v_layers, k_out_layers, v_out_layers, win_idx, tok_idx, n_keep, workspace, stream)
PyObject *compress_group(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *q, *lse, *t[3], *ws, *st;
  size_t bytes;
  int32_t gamma;
  Pointers<WKV_MAX_LAYERS> k, v, ko, vo;
  if (!arity(n, 13) || !pr.fill(a[0], problem_kind) || !integer(a[1], &gamma) || !pointer(a[2], &q) || !pointer(a[3], &lse) || !k.fill(a[4]) ||
      !v.fill(a[5]) || !ko.fill(a[6]) || !vo.fill(a[7])) return nullptr;
  for (int i = 0; i < 3; ++i) if (!pointer(a[8 + i], &t[i])) return nullptr;
  if (!workspace(a[11], &ws, &bytes) || !stream_of(a[12], &st)) return nullptr;
  return call([&] {
    return wkv_compress_group(pr.problem(), gamma, q, (const float *)lse, k.p, v.p, ko.p, vo.p, (int32_t *)t[0], (int32_t *)t[1],
                              (int32_t *)t[2], ws, bytes, st);
  });
}

// (problem, n_groups, gamma, q_obs_groups, lse_obs_groups | None, k_windows_groups | None (nested), k_layers, v_layers,
//  k_out_layers, v_out_layers, win_idx, tok_idx, n_keep, workspace, stream)
PyObject *compress_groups(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Structure pr;
  void *t[3], *ws, *st;
  size_t bytes;
  int32_t n_groups, gamma;
  Pointers<WKV_MAX_LAYERS> k, v, ko, vo;
  Pointers<WKV_MAX_GROUPS> q, lse;
  int32_t budgets[WKV_MAX_GROUPS * WKV_MAX_BATCH];
  if (!arity(n, 15) || !pr.fill(a[0], problem_kind) || !integer(a[1], &n_groups) || !integer(a[2], &gamma) || !q.fill(a[3])) return nullptr;
  if (a[4] != Py_None && !lse.fill(a[4])) return nullptr;
  if (a[5] != Py_None) {                     // row-major, as the ABI wants it; entries a caller leaves out are -1: refused
    std::memset(budgets, 0xff, sizeof budgets);
    PyObject *rows = PySequence_Fast(a[5], "k_windows_groups: expected [n_groups][batch] integers");
    if (!rows) return nullptr;
    Py_ssize_t at = 0;
    bool ok = true;
    for (Py_ssize_t g = 0; ok && g < PySequence_Fast_GET_SIZE(rows); ++g) {
      PyObject *row = PySequence_Fast(PySequence_Fast_GET_ITEM(rows, g), "k_windows_groups: expected [n_groups][batch] integers");
      ok = row != nullptr;
      for (Py_ssize_t b = 0; ok && b < PySequence_Fast_GET_SIZE(row) && at < WKV_MAX_GROUPS * WKV_MAX_BATCH; ++b, ++at) {
        PyObject *i = PyNumber_Long(PySequence_Fast_GET_ITEM(row, b));
        ok = i && integer(i, &budgets[at]);
        Py_XDECREF(i);
      }
      Py_XDECREF(row);
    }
    Py_DECREF(rows);
    if (!ok) return nullptr;
  }
  if (!k.fill(a[6]) || !v.fill(a[7]) || !ko.fill(a[8]) || !vo.fill(a[9])) return nullptr;
  for (int i = 0; i < 3; ++i) if (!pointer(a[10 + i], &t[i])) return nullptr;
  if (!workspace(a[13], &ws, &bytes) || !stream_of(a[14], &st)) return nullptr;
  return call([&] {
    return wkv_compress_groups(pr.problem(), n_groups, gamma, q.p, a[4] == Py_None ? nullptr : (const float *const *)lse.p,
                               a[5] == Py_None ? nullptr : budgets, k.p, v.p, ko.p, vo.p, (int32_t *)t[0], (int32_t *)t[1],
                               (int32_t *)t[2], ws, bytes, st);
  });
}

// (slow_stream, convert, Problem, its structure, DecodeShape, its structure)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 6)) return nullptr;
  PyObject **to[6] = {&slow_stream, &convert, &problem_kind.wrapper, &problem_kind.structure, &shape_kind.wrapper, &shape_kind.structure};
  for (int i = 0; i < 6; ++i) {
    Py_INCREF(a[i]);
    Py_XSETREF(*to[i], a[i]);
  }
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(decode_step), FAST(decode_step_static), FAST(score), FAST(window_pool), FAST(topk_windows),
                         FAST(gather_group), FAST(compress_group), FAST(compress_groups),
                         FAST(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  s_c = PyUnicode_InternFromString("c");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  if (!s_c || !s_data_ptr || !s_numel || !s_element_size) return nullptr;
  return PyModule_Create(&module);
}
