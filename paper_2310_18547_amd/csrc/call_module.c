// CPython module with the calls a decode loop makes once per layer and projection.
//
// What bounds it: a decode add-on runs 4-6 us on the GPU, and one call through ctypes cost the
// host 5.3 us, of which 3.4 us are the kernel launch itself -- the loop was bound by its host
// side.  ctypes spends 1.1 us on converting the arguments and Python code another 0.7 us on
// taking the tensors' addresses; here both are done in C from the interpreter's argument vector
// (vectorcall, nothing is packed into tuples or dicts).  The functions keep the names, argument
// order, keywords, defaults, results and exceptions they had as Python code.
//
// The module calls the library that binding.py has loaded: it is handed the entry points'
// addresses, so that a tuning build of the library works the same way.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/sgmv.h"

typedef int (*shrink_fn)(const sgmv_problem*, float*, const void*, const void* const*, const int32_t*, int32_t, int32_t,
                         void*);
typedef int (*expand_fn)(const sgmv_problem*, void*, const float*, const void* const*, const int32_t*, int32_t, int32_t,
                         float, void*);
typedef int (*add_lora_fn)(const sgmv_problem*, void*, const void*, const void* const*, const void* const*,
                           const int32_t*, int32_t, int32_t, float, void*);
typedef int (*add_lora_multi_fn)(const sgmv_problem*, int32_t, void* const*, const void* const*,
                                 const void* const* const*, const void* const* const*, const int32_t*, int32_t,
                                 int32_t, float, void*);

static shrink_fn fn_shrink;
static expand_fn fn_expand;
static add_lora_fn fn_add_lora;
static add_lora_fn fn_add_lora_static;
static add_lora_multi_fn fn_add_lora_multi;
static PyObject* problem_type;  // binding.SgmvProblem
static PyObject* error_type;    // binding.SgmvError
static PyObject *str_data_ptr, *str_ctypes, *str_data, *str_cuda_stream;

// The address behind a pointer argument: None, an int, or an object with data_ptr() (a tensor) or
// ctypes.data (a numpy array).  0 on success.
static int address_of(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = NULL;
    return 0;
  }
  PyObject* value;
  if (PyLong_Check(o)) {
    value = o;
    Py_INCREF(value);
  } else {
    value = PyObject_CallMethodNoArgs(o, str_data_ptr);
    if (value == NULL) {
      if (!PyErr_ExceptionMatches(PyExc_AttributeError) || PyObject_HasAttr(o, str_data_ptr)) return -1;
      PyErr_Clear();
      PyObject* c = PyObject_GetAttr(o, str_ctypes);
      if (c == NULL) {
        if (PyErr_ExceptionMatches(PyExc_AttributeError)) {
          PyErr_Clear();
          PyErr_Format(PyExc_TypeError, "cannot take the address of %R", (PyObject*)Py_TYPE(o));
        }
        return -1;
      }
      value = PyObject_GetAttr(c, str_data);
      Py_DECREF(c);
      if (value == NULL) return -1;
    }
  }
  const unsigned long long a = PyLong_AsUnsignedLongLongMask(value);
  Py_DECREF(value);
  if (a == (unsigned long long)-1 && PyErr_Occurred()) return -1;
  *out = (void*)(uintptr_t)a;
  return 0;
}

// None, an int, or an object with cuda_stream (a torch stream).
static int stream_of(PyObject* o, void** out) {
  if (o == NULL || o == Py_None || PyLong_Check(o)) return address_of(o == NULL ? Py_None : o, out);
  PyObject* s = PyObject_GetAttr(o, str_cuda_stream);
  if (s == NULL) return -1;
  const int rc = address_of(s, out);
  Py_DECREF(s);
  return rc;
}

static int int32_of(PyObject* o, int32_t* out) {
  const unsigned long v = PyLong_AsUnsignedLongMask(o);  // takes __index__, wraps like a C cast
  if (v == (unsigned long)-1 && PyErr_Occurred()) return -1;
  *out = (int32_t)v;
  return 0;
}

static int float_of(PyObject* o, float* out) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) return -1;
  *out = (float)v;
  return 0;
}

// The caller's struct sgmv_problem; PyBuffer_Release when done.
static int problem_of(PyObject* o, Py_buffer* view) {
  const int is = PyObject_IsInstance(o, problem_type);
  if (is < 0) return -1;
  if (!is) {
    PyErr_Format(PyExc_TypeError, "expected an SgmvProblem, got %R", (PyObject*)Py_TYPE(o));
    return -1;
  }
  return PyObject_GetBuffer(o, view, PyBUF_SIMPLE);
}

// Positional and keyword arguments into `got` by name; the first `required` must be there.
static int sort_arguments(const char* where, const char* const* names, int n, int required, PyObject* const* args,
                          Py_ssize_t nargs, PyObject* kwnames, PyObject** got) {
  if (nargs > n) {
    PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", where, n, nargs);
    return -1;
  }
  for (int i = 0; i < n; ++i) got[i] = i < nargs ? args[i] : NULL;
  const Py_ssize_t nkw = kwnames == NULL ? 0 : PyTuple_GET_SIZE(kwnames);
  for (Py_ssize_t k = 0; k < nkw; ++k) {
    PyObject* key = PyTuple_GET_ITEM(kwnames, k);
    int i = 0;
    while (i < n && PyUnicode_CompareWithASCIIString(key, names[i]) != 0) ++i;
    if (i == n) {
      PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", where, key);
      return -1;
    }
    if (got[i] != NULL) {
      PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", where, key);
      return -1;
    }
    got[i] = args[nargs + k];
  }
  for (int i = 0; i < required; ++i) {
    if (got[i] == NULL) {
      PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", where, names[i]);
      return -1;
    }
  }
  return 0;
}

// The call's status as a Python int, or SgmvError(status, where) when `check` is true (the default).
static PyObject* finish(int rc, PyObject* check, const char* where) {
  if (rc != 0) {
    const int raise = check == NULL ? 1 : PyObject_IsTrue(check);
    if (raise < 0) return NULL;
    if (raise) {
      PyObject* e = PyObject_CallFunction(error_type, "is", rc, where);
      if (e != NULL) {
        PyErr_SetObject(error_type, e);
        Py_DECREF(e);
      }
      return NULL;
    }
  }
  return PyLong_FromLong(rc);
}

static PyObject* call_shrink(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p", "v", "x", "A_ptrs", "seg_starts", "n_segs", "layer_idx", "stream", "check"};
  PyObject* g[9];
  if (sort_arguments("sgmv_shrink", names, 9, 7, args, nargs, kwnames, g) < 0) return NULL;
  void *v, *x, *a, *seg, *stream;
  int32_t n_segs, layer;
  if (address_of(g[1], &v) < 0 || address_of(g[2], &x) < 0 || address_of(g[3], &a) < 0 || address_of(g[4], &seg) < 0 ||
      int32_of(g[5], &n_segs) < 0 || int32_of(g[6], &layer) < 0 || stream_of(g[7], &stream) < 0)
    return NULL;
  Py_buffer p;
  if (problem_of(g[0], &p) < 0) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn_shrink((const sgmv_problem*)p.buf, (float*)v, x, (const void* const*)a, (const int32_t*)seg, n_segs, layer, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[8], "sgmv_shrink");
}

static PyObject* call_expand(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p", "y", "v", "B_ptrs", "seg_starts", "n_segs", "layer_idx", "scale", "stream", "check"};
  PyObject* g[10];
  if (sort_arguments("sgmv_expand", names, 10, 8, args, nargs, kwnames, g) < 0) return NULL;
  void *y, *v, *b, *seg, *stream;
  int32_t n_segs, layer;
  float scale;
  if (address_of(g[1], &y) < 0 || address_of(g[2], &v) < 0 || address_of(g[3], &b) < 0 || address_of(g[4], &seg) < 0 ||
      int32_of(g[5], &n_segs) < 0 || int32_of(g[6], &layer) < 0 || float_of(g[7], &scale) < 0 ||
      stream_of(g[8], &stream) < 0)
    return NULL;
  Py_buffer p;
  if (problem_of(g[0], &p) < 0) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn_expand((const sgmv_problem*)p.buf, y, (const float*)v, (const void* const*)b, (const int32_t*)seg, n_segs, layer,
                 scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[9], "sgmv_expand");
}

static PyObject* add_lora(add_lora_fn fn, const char* where, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p",      "y",         "x",     "A_ptrs", "B_ptrs", "seg_starts",
                                      "n_segs", "layer_idx", "scale", "stream", "check"};
  PyObject* g[11];
  if (sort_arguments(where, names, 11, 9, args, nargs, kwnames, g) < 0) return NULL;
  void *y, *x, *a, *b, *seg, *stream;
  int32_t n_segs, layer;
  float scale;
  if (address_of(g[1], &y) < 0 || address_of(g[2], &x) < 0 || address_of(g[3], &a) < 0 || address_of(g[4], &b) < 0 ||
      address_of(g[5], &seg) < 0 || int32_of(g[6], &n_segs) < 0 || int32_of(g[7], &layer) < 0 ||
      float_of(g[8], &scale) < 0 || stream_of(g[9], &stream) < 0)
    return NULL;
  Py_buffer p;
  if (problem_of(g[0], &p) < 0) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn((const sgmv_problem*)p.buf, y, x, (const void* const*)a, (const void* const*)b, (const int32_t*)seg, n_segs,
          layer, scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[10], where);
}

static PyObject* call_add_lora(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  return add_lora(fn_add_lora, "sgmv_add_lora", args, nargs, kwnames);
}

static PyObject* call_add_lora_static(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  return add_lora(fn_add_lora_static, "sgmv_add_lora_static", args, nargs, kwnames);
}

// The addresses of a sequence's `n` elements; more than the library takes are left for it to refuse.
// An element's data_ptr() is Python code and may change the very list that is read: the size is looked up
// again and the element kept alive around each one, and what is no longer there counts as NULL.
#define MOST_ADD_ONS 64
static int addresses_of(PyObject* seq, Py_ssize_t n, void** out) {
  PyObject* fast = PySequence_Fast(seq, "expected a sequence");
  if (fast == NULL) return -1;
  int rc = 0;
  if (PySequence_Fast_GET_SIZE(fast) != n) {
    PyErr_SetString(PyExc_IndexError, "sequences of pointers differ in length");
    rc = -1;
  }
  for (Py_ssize_t i = 0; i < n && rc == 0; ++i) {
    out[i] = NULL;
    if (i >= PySequence_Fast_GET_SIZE(fast)) continue;
    PyObject* element = PySequence_Fast_GET_ITEM(fast, i);
    Py_INCREF(element);
    rc = address_of(element, &out[i]);
    Py_DECREF(element);
  }
  Py_DECREF(fast);
  return rc;
}

static PyObject* call_add_lora_multi(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p",      "ys",        "xs",    "A_ptrs", "B_ptrs", "seg_starts",
                                      "n_segs", "layer_idx", "scale", "stream", "check"};
  static const char where[] = "sgmv_add_lora_multi";
  PyObject* g[11];
  if (sort_arguments(where, names, 11, 9, args, nargs, kwnames, g) < 0) return NULL;
  const Py_ssize_t n = PySequence_Size(g[1]);
  if (n < 0) return NULL;
  if (n > MOST_ADD_ONS) return finish(SGMV_ERR_SHAPE, g[10], where);
  void *ys[MOST_ADD_ONS], *xs[MOST_ADD_ONS], *as[MOST_ADD_ONS], *bs[MOST_ADD_ONS], *seg, *stream;
  int32_t n_segs, layer;
  float scale;
  if (addresses_of(g[1], n, ys) < 0 || addresses_of(g[2], n, xs) < 0 || addresses_of(g[3], n, as) < 0 ||
      addresses_of(g[4], n, bs) < 0 || address_of(g[5], &seg) < 0 || int32_of(g[6], &n_segs) < 0 ||
      int32_of(g[7], &layer) < 0 || float_of(g[8], &scale) < 0 || stream_of(g[9], &stream) < 0)
    return NULL;
  Py_buffer p;
  if (problem_of(g[0], &p) < 0) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn_add_lora_multi((const sgmv_problem*)p.buf, (int32_t)n, ys, (const void* const*)xs, (const void* const* const*)as,
                         (const void* const* const*)bs, (const int32_t*)seg, n_segs, layer, scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[10], where);
}

// bind(problem type, error type, addresses of sgmv_shrink, sgmv_expand, sgmv_add_lora,
// sgmv_add_lora_static and sgmv_add_lora_multi)
static PyObject* call_bind(PyObject* self, PyObject* args) {
  PyObject *problem, *error;
  unsigned long long f[5];
  if (!PyArg_ParseTuple(args, "OOKKKKK", &problem, &error, &f[0], &f[1], &f[2], &f[3], &f[4])) return NULL;
  Py_INCREF(problem);
  Py_INCREF(error);
  Py_XSETREF(problem_type, problem);
  Py_XSETREF(error_type, error);
  fn_shrink = (shrink_fn)(uintptr_t)f[0];
  fn_expand = (expand_fn)(uintptr_t)f[1];
  fn_add_lora = (add_lora_fn)(uintptr_t)f[2];
  fn_add_lora_static = (add_lora_fn)(uintptr_t)f[3];
  fn_add_lora_multi = (add_lora_multi_fn)(uintptr_t)f[4];
  return PyLong_FromSize_t(sizeof(sgmv_problem));
}

#define FAST(name, fn, doc) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL | METH_KEYWORDS, doc}
static PyMethodDef methods[] = {
    FAST("sgmv_shrink", call_shrink,
         "sgmv_shrink(p, v, x, A_ptrs, seg_starts, n_segs, layer_idx, stream=None, check=True)\n--\n\n"),
    FAST("sgmv_expand", call_expand,
         "sgmv_expand(p, y, v, B_ptrs, seg_starts, n_segs, layer_idx, scale, stream=None, check=True)\n--\n\n"),
    FAST("sgmv_add_lora", call_add_lora,
         "sgmv_add_lora(p, y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, scale, stream=None, check=True)\n--\n\n"),
    FAST("sgmv_add_lora_static", call_add_lora_static,
         "sgmv_add_lora_static(p, y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, scale, stream=None, check=True)\n--\n\n"),
    FAST("sgmv_add_lora_multi", call_add_lora_multi,
         "sgmv_add_lora_multi(p, ys, xs, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, scale, stream=None, check=True)\n"
         "--\n\nys, xs, A_ptrs, B_ptrs are sequences of equal length (one entry per add-on)."),
    {"bind", call_bind, METH_VARARGS, "bind(problem_type, error_type, *entry_points) -> size of the C struct"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sgmv_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__sgmv_call(void) {
  str_data_ptr = PyUnicode_InternFromString("data_ptr");
  str_ctypes = PyUnicode_InternFromString("ctypes");
  str_data = PyUnicode_InternFromString("data");
  str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!str_data_ptr || !str_ctypes || !str_data || !str_cuda_stream) return NULL;
  return PyModule_Create(&module);
}
