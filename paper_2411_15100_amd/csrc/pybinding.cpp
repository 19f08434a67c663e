// The per-step calls of the Python binding as a CPython extension (_native):
// accepting tokens, fills, applies, device-batch steps.  Marshalling only, as
// in binding.py, which installs these functions when it loads libxgm.so and
// hands over the addresses of the entry points (so that this file links to
// nothing).  A call costs 0.1 us of Python this way; through ctypes it was 0.5
// us for a token and 1.2 us for a launch, as much as the work itself: a step of
// 32 host matchers spent 14 of its 20 us there.  Every call lets other threads
// run, as through ctypes, which costs 0.06 us (16 steps of 32 rows: 151 -> 160).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>

namespace {

struct {
  const char* (*last_error)();
  int (*matcher_accept_token)(void*, int32_t);
  int (*matcher_accept_bytes)(void*, const uint8_t*, int32_t);
  int (*matcher_reset)(void*);
  int (*fill_next_token_bitmask)(void* const*, int32_t, void*, void*);
  int (*fill_next_token_bitmask_static)(void* const*, int32_t, void*, void*);
  int (*fill_and_apply)(void* const*, int32_t, void*, void*, int, int32_t, int64_t, void*);
  int (*apply_token_bitmask_inplace)(void*, int, int32_t, int32_t, int64_t, const void*, int32_t, const void*, int32_t, void*);
  int (*batch_accept_tokens)(void*, const void*, void*);
  int (*batch_rollback)(void*, const void*, void*);
  int (*batch_fork)(void*, const void*, void*);
  int (*batch_fill_next_token_bitmask)(void*, void*, void*);
  int (*batch_fill_and_apply)(void*, void*, void*, int, int32_t, int64_t, void*);
} api;
struct { const char* name; void** slot; } const kEntries[] = {
    {"xgm_last_error", (void**)&api.last_error},
    {"xgm_matcher_accept_token", (void**)&api.matcher_accept_token},
    {"xgm_matcher_accept_bytes", (void**)&api.matcher_accept_bytes},
    {"xgm_matcher_reset", (void**)&api.matcher_reset},
    {"xgm_fill_next_token_bitmask", (void**)&api.fill_next_token_bitmask},
    {"xgm_fill_next_token_bitmask_static", (void**)&api.fill_next_token_bitmask_static},
    {"xgm_fill_and_apply", (void**)&api.fill_and_apply},
    {"xgm_apply_token_bitmask_inplace", (void**)&api.apply_token_bitmask_inplace},
    {"xgm_batch_accept_tokens", (void**)&api.batch_accept_tokens},
    {"xgm_batch_rollback", (void**)&api.batch_rollback},
    {"xgm_batch_fork", (void**)&api.batch_fork},
    {"xgm_batch_fill_next_token_bitmask", (void**)&api.batch_fill_next_token_bitmask},
    {"xgm_batch_fill_and_apply", (void**)&api.batch_fill_and_apply},
};
PyObject* g_error_class = nullptr;  // XgmError(status, message)
PyObject *s_h, *s_addr, *s_matchers;

PyObject* result(int rc) {
  if (rc >= 0) Py_RETURN_NONE;
  PyObject* msg = PyUnicode_DecodeUTF8(api.last_error(), (Py_ssize_t)strlen(api.last_error()), "replace");
  if (!msg) return nullptr;
  PyObject* e = PyObject_CallFunction(g_error_class, "iN", rc, msg);
  if (e) {
    PyErr_SetObject(g_error_class, e);
    Py_DECREF(e);
  }
  return nullptr;
}

// the arguments by position or by name; absent ones are null (the first `required` must be there)
template <int N>
bool arguments(const char* fn, PyObject* const* args, Py_ssize_t n, PyObject* kwnames, const char* const (&names)[N], int required,
               PyObject* (&out)[N]) {
  for (int k = 0; k < N; ++k) out[k] = k < n ? args[k] : nullptr;
  if (n > N) { PyErr_Format(PyExc_TypeError, "%s() takes %d arguments (%zd given)", fn, N, n); return false; }
  for (Py_ssize_t j = 0; kwnames && j < PyTuple_GET_SIZE(kwnames); ++j) {
    PyObject* name = PyTuple_GET_ITEM(kwnames, j);
    int k = 0;
    while (k < N && PyUnicode_CompareWithASCIIString(name, names[k]) != 0) ++k;
    if (k == N) { PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", fn, name); return false; }
    if (out[k]) { PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", fn, name); return false; }
    out[k] = args[n + j];
  }
  for (int k = 0; k < required; ++k)
    if (!out[k]) { PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", fn, names[k]); return false; }
  return true;
}
bool low_bits(PyObject* o, int64_t* out) {
  *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
  return *out != -1 || !PyErr_Occurred();
}
bool converted(PyObject* v, int64_t* out) {  // (takes over v)
  const bool ok = v && low_bits(v, out);
  Py_XDECREF(v);
  return ok;
}
// an address: an integer, or None (or absent) for null
bool address(PyObject* o, int64_t* out) {
  if (!o || o == Py_None) { *out = 0; return true; }
  return PyLong_Check(o) ? low_bits(o, out) : converted(PyNumber_Index(o), out);
}
bool integer(PyObject* o, int64_t* out) { return PyLong_Check(o) ? low_bits(o, out) : converted(PyNumber_Index(o), out); }
// a number, as int() takes it
bool number(PyObject* o, int64_t* out) { return PyLong_Check(o) ? low_bits(o, out) : converted(PyNumber_Long(o), out); }
// kinds[k]: 'a' for an address, 'n' for a number, 'i' for an integer
template <int N>
bool values(PyObject* const* in, int64_t (&out)[N], const char (&kinds)[N + 1]) {
  for (int k = 0; k < N; ++k)
    if (!(kinds[k] == 'a' ? address(in[k], &out[k]) : kinds[k] == 'n' ? number(in[k], &out[k]) : integer(in[k], &out[k]))) return false;
  return true;
}
void* pointer(int64_t v) { return reinterpret_cast<void*>((uintptr_t)v); }
bool attribute(PyObject* self, PyObject* name, void** out) {
  PyObject* h = PyObject_GetAttr(self, name);
  if (!h) return false;
  int64_t v = 0;
  const bool ok = address(h, &v);
  Py_DECREF(h);
  *out = pointer(v);
  return ok;
}

// ---- methods of Matcher
PyObject* matcher_accept_token(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"token_id"};
  PyObject* a[1];
  int64_t v[1];
  void* h;
  if (!arguments("accept_token", args, n, kwnames, names, 1, a) || !values(a, v, "n") || !attribute(self, s_h, &h)) return nullptr;
  int rc;  // (a token of an ambiguous grammar, or a long one, may take milliseconds)
  Py_BEGIN_ALLOW_THREADS
  rc = api.matcher_accept_token(h, (int32_t)v[0]);
  Py_END_ALLOW_THREADS
  return result(rc);
}
PyObject* matcher_accept_bytes(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"data"};
  PyObject* a[1];
  char* bytes;
  Py_ssize_t len;
  void* h;
  if (!arguments("accept_bytes", args, n, kwnames, names, 1, a) || PyBytes_AsStringAndSize(a[0], &bytes, &len) < 0 || !attribute(self, s_h, &h))
    return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.matcher_accept_bytes(h, (const uint8_t*)bytes, (int32_t)len);
  Py_END_ALLOW_THREADS
  return result(rc);
}
PyObject* matcher_reset(PyObject* self, PyObject*) {
  void* h;
  if (!attribute(self, s_h, &h)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.matcher_reset(h);
  Py_END_ALLOW_THREADS
  return result(rc);
}

// ---- methods of DeviceBatch
PyObject* batch_step(PyObject* self, int (*step)(void*, const void*, void*), const char* fn, const char* const (&names)[2], PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  PyObject* a[2];
  int64_t v[2];
  void* h;
  if (!arguments(fn, args, n, kwnames, names, 1, a) || !values(a, v, "aa") || !attribute(self, s_h, &h)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = step(h, pointer(v[0]), pointer(v[1]));
  Py_END_ALLOW_THREADS
  return result(rc);
}
PyObject* batch_accept_tokens(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"d_token_ids", "stream"};
  return batch_step(self, api.batch_accept_tokens, "accept_tokens", names, args, n, kwnames);
}
PyObject* batch_rollback(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"d_steps", "stream"};
  return batch_step(self, api.batch_rollback, "rollback", names, args, n, kwnames);
}
PyObject* batch_fork(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"d_src_rows", "stream"};
  return batch_step(self, api.batch_fork, "fork", names, args, n, kwnames);
}
PyObject* batch_fill(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"d_bitmask", "stream"};
  PyObject* a[2];
  int64_t v[2];
  void* h;
  if (!arguments("fill_next_token_bitmask", args, n, kwnames, names, 1, a) || !values(a, v, "aa") || !attribute(self, s_h, &h)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.batch_fill_next_token_bitmask(h, pointer(v[0]), pointer(v[1]));
  Py_END_ALLOW_THREADS
  return result(rc);
}
PyObject* batch_fill_and_apply(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
  static const char* const names[] = {"d_bitmask", "d_logits", "dtype", "v_logits", "row_stride", "stream"};
  PyObject* a[6];
  int64_t v[6];
  void* h;
  if (!arguments("fill_and_apply", args, n, kwnames, names, 5, a) || !values(a, v, "aannna") || !attribute(self, s_h, &h)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.batch_fill_and_apply(h, pointer(v[0]), pointer(v[1]), (int)v[2], (int32_t)v[3], v[4], pointer(v[5]));
  Py_END_ALLOW_THREADS
  return result(rc);
}

// ---- functions over matchers
// The handles of a MatcherBatch (prepared once) or of a sequence of matchers, which are kept alive for the call: other
// threads run meanwhile, and a sequence may be the only one that has them.
class Handles {
 public:
  bool get(PyObject* matchers) {
    PyObject* list = PyObject_GetAttr(matchers, s_matchers);
    if (list) {
      n_ = PyObject_Length(list);
      Py_DECREF(list);
      void* p = nullptr;
      if (n_ < 0 || !attribute(matchers, s_addr, &p)) return false;
      data_ = (void**)p;
      return true;
    }
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
    PyErr_Clear();
    kept_ = PySequence_Tuple(matchers);
    if (!kept_) return false;
    n_ = PyTuple_GET_SIZE(kept_);
    void** p = few_;
    if (n_ > kFew) p = own_ = (void**)PyMem_Malloc(sizeof(void*) * (size_t)n_);
    bool ok = p != nullptr;
    if (!ok) PyErr_NoMemory();
    for (Py_ssize_t k = 0; ok && k < n_; ++k) ok = attribute(PyTuple_GET_ITEM(kept_, k), s_h, &p[k]);
    data_ = p;
    return ok;
  }
  ~Handles() {
    PyMem_Free(own_);
    Py_XDECREF(kept_);
  }
  void* const* data() const { return data_; }
  int32_t size() const { return (int32_t)n_; }

 private:
  static constexpr Py_ssize_t kFew = 256;
  PyObject* kept_ = nullptr;
  void* few_[kFew];
  void** own_ = nullptr;
  void** data_ = nullptr;
  Py_ssize_t n_ = 0;
};
// fill_next_token_bitmask(matchers, d_bitmask, stream, static)
PyObject* fill(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 4) return PyErr_Format(PyExc_TypeError, "fill takes 4 arguments");
  int64_t v[2];
  Handles h;
  if (!h.get(args[0]) || !values(args + 1, v, "aa")) return nullptr;
  auto fn = args[3] == Py_True ? api.fill_next_token_bitmask_static : api.fill_next_token_bitmask;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(h.data(), h.size(), pointer(v[0]), pointer(v[1]));
  Py_END_ALLOW_THREADS
  return result(rc);
}
// fill_and_apply(matchers, d_bitmask, d_logits, dtype, v_logits, row_stride, stream)
PyObject* fill_and_apply(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 7) return PyErr_Format(PyExc_TypeError, "fill_and_apply takes 7 arguments");
  int64_t v[6];
  Handles h;
  if (!h.get(args[0]) || !values(args + 1, v, "aannna")) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.fill_and_apply(h.data(), h.size(), pointer(v[0]), pointer(v[1]), (int)v[2], (int32_t)v[3], v[4], pointer(v[5]));
  Py_END_ALLOW_THREADS
  return result(rc);
}
// apply_token_bitmask_inplace(d_logits, dtype, B, V_logits, row_stride, d_bitmask, V_mask, d_row_index, n_rows, stream)
PyObject* apply(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 10) return PyErr_Format(PyExc_TypeError, "apply takes 10 arguments");
  int64_t v[10];
  if (!values(args, v, "aiiiiaiaia")) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = api.apply_token_bitmask_inplace(pointer(v[0]), (int)v[1], (int32_t)v[2], (int32_t)v[3], v[4], pointer(v[5]), (int32_t)v[6], pointer(v[7]),
                                       (int32_t)v[8], pointer(v[9]));
  Py_END_ALLOW_THREADS
  return result(rc);
}

#define FAST(fn) (PyCFunction)(void (*)(void))(fn), METH_FASTCALL
#define FAST_KW(fn) (PyCFunction)(void (*)(void))(fn), METH_FASTCALL | METH_KEYWORDS
PyMethodDef kMatcherMethods[] = {
    {"accept_token", FAST_KW(matcher_accept_token), "accept_token(token_id): the token joins the text"},
    {"accept_bytes", FAST_KW(matcher_accept_bytes), "accept_bytes(data): the bytes join the text"},
    {"reset", matcher_reset, METH_NOARGS, "reset(): back to the empty text"},
};
PyMethodDef kBatchMethods[] = {
    {"accept_tokens", FAST_KW(batch_accept_tokens), "accept_tokens(d_token_ids, stream=0)"},
    {"rollback", FAST_KW(batch_rollback), "rollback(d_steps, stream=0)"},
    {"fork", FAST_KW(batch_fork), "fork(d_src_rows, stream=0)"},
    {"fill_next_token_bitmask", FAST_KW(batch_fill), "fill_next_token_bitmask(d_bitmask, stream=0)"},
    {"fill_and_apply", FAST_KW(batch_fill_and_apply), "fill_and_apply(d_bitmask, d_logits, dtype, v_logits, row_stride, stream=0)"},
};
template <size_t N>
bool put_methods(PyObject* cls, PyMethodDef (&defs)[N]) {
  for (auto& d : defs) {
    PyObject* m = PyDescr_NewMethod((PyTypeObject*)cls, &d);
    if (!m) return false;
    const int rc = PyObject_SetAttrString(cls, d.ml_name, m);
    Py_DECREF(m);
    if (rc < 0) return false;
  }
  return true;
}
// install(addresses, XgmError, Matcher, DeviceBatch): addresses[name] = address of the entry point
PyObject* install(PyObject*, PyObject* args) {
  PyObject *addresses, *error, *matcher, *batch;
  if (!PyArg_ParseTuple(args, "O!OO!O!", &PyDict_Type, &addresses, &error, &PyType_Type, &matcher, &PyType_Type, &batch)) return nullptr;
  for (auto& e : kEntries) {
    PyObject* a = PyDict_GetItemString(addresses, e.name);
    if (!a) return PyErr_Format(PyExc_KeyError, "no address of %s", e.name);
    if (!(*e.slot = PyLong_AsVoidPtr(a))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "null address of %s", e.name);
  }
  Py_INCREF(error);
  Py_XSETREF(g_error_class, error);
  if (!put_methods(matcher, kMatcherMethods) || !put_methods(batch, kBatchMethods)) return nullptr;
  Py_RETURN_NONE;
}
PyMethodDef kFunctions[] = {
    {"install", install, METH_VARARGS, nullptr},
    {"fill", FAST(fill), nullptr},
    {"fill_and_apply", FAST(fill_and_apply), nullptr},
    {"apply", FAST(apply), nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "the per-step calls of binding.py", -1, kFunctions, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  s_h = PyUnicode_InternFromString("_h");
  s_addr = PyUnicode_InternFromString("_addr");
  s_matchers = PyUnicode_InternFromString("matchers");
  if (!s_h || !s_addr || !s_matchers) return nullptr;
  return PyModule_Create(&kModule);
}
