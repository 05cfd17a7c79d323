// CPython module with the calls a decode loop makes once per layer and projection.
//
// What bounds it: a decode add-on runs 4-6 us on the GPU, and one call through ctypes cost the
// host 5.3 us, of which 3.4 us are the kernel launch itself -- the loop was bound by its host
// side.  ctypes spends 1.1 us on converting the arguments and Python code another 0.7 us on
// taking the tensors' addresses; here both are done in C from the interpreter's argument vector
// (vectorcall, nothing is packed into tuples or dicts).
//
// Only the usual forms are converted here: addresses as ints, None or objects with data_ptr(), numbers
// as Python converts them, lists or tuples of pointers.  A call with anything else in it (ctypes objects,
// numpy arrays, pointer lists of different lengths, wrong arguments) goes, arguments untouched, to the
// Python function of the same name in binding.py, whose answer or exception it gets.
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
static PyObject* general[5];    // the functions in Python, in the order of bind()'s addresses
enum { SHRINK, EXPAND, ADD_LORA, ADD_LORA_STATIC, ADD_LORA_MULTI };
static PyObject *str_data_ptr, *str_cuda_stream;

// What the conversions below return besides an error (-1, an exception is set): the value is there, or
// the argument is not of a usual form.
enum { DONE = 0, UNUSUAL = 1 };

// After a failed conversion: the general function decides what becomes of the argument.
static int unusual(void) {
  if (!PyErr_ExceptionMatches(PyExc_Exception)) return -1;  // an interrupt stays one
  PyErr_Clear();
  return UNUSUAL;
}

// The address behind a pointer argument: None, an int, or an object with data_ptr() (a tensor).
static int address_of(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = NULL;
    return DONE;
  }
  PyObject* value;
  if (PyLong_Check(o)) {
    value = o;
    Py_INCREF(value);
  } else {
    value = PyObject_CallMethodNoArgs(o, str_data_ptr);
    if (value == NULL) return unusual();
  }
  int rc = UNUSUAL;
  if (PyLong_Check(value)) {
    const unsigned long long a = PyLong_AsUnsignedLongLongMask(value);
    rc = a == (unsigned long long)-1 && PyErr_Occurred() ? unusual() : DONE;
    *out = (void*)(uintptr_t)a;
  }
  Py_DECREF(value);
  return rc;
}

// None, an int, or an object with cuda_stream (a torch stream).
static int stream_of(PyObject* o, void** out) {
  if (o == NULL || o == Py_None || PyLong_Check(o)) return address_of(o == NULL ? Py_None : o, out);
  PyObject* s = PyObject_GetAttr(o, str_cuda_stream);
  if (s == NULL) return unusual();
  const int rc = s == Py_None || PyLong_Check(s) ? address_of(s, out) : UNUSUAL;
  Py_DECREF(s);
  return rc;
}

static int int32_of(PyObject* o, int32_t* out) {
  if (!PyIndex_Check(o)) return UNUSUAL;
  const unsigned long v = PyLong_AsUnsignedLongMask(o);  // wraps like a C cast
  if (v == (unsigned long)-1 && PyErr_Occurred()) return unusual();
  *out = (int32_t)v;
  return DONE;
}

static int float_of(PyObject* o, float* out) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) return unusual();
  *out = (float)v;
  return DONE;
}

// The caller's struct sgmv_problem; PyBuffer_Release when done.
static int problem_of(PyObject* o, Py_buffer* view) {
  const int is = PyObject_IsInstance(o, problem_type);
  if (is < 0) return -1;
  if (!is) return UNUSUAL;
  return PyObject_GetBuffer(o, view, PyBUF_SIMPLE);
}

// Positional and keyword arguments into `got` by name; the first `required` must be there.
static int sort_arguments(const char* const* names, int n, int required, PyObject* const* args, Py_ssize_t nargs,
                          PyObject* kwnames, PyObject** got) {
  if (nargs > n) return UNUSUAL;
  for (int i = 0; i < n; ++i) got[i] = i < nargs ? args[i] : NULL;
  const Py_ssize_t nkw = kwnames == NULL ? 0 : PyTuple_GET_SIZE(kwnames);
  for (Py_ssize_t k = 0; k < nkw; ++k) {
    PyObject* key = PyTuple_GET_ITEM(kwnames, k);
    int i = 0;
    while (i < n && PyUnicode_CompareWithASCIIString(key, names[i]) != 0) ++i;
    if (i == n || got[i] != NULL) return UNUSUAL;
    got[i] = args[nargs + k];
  }
  for (int i = 0; i < required; ++i)
    if (got[i] == NULL) return UNUSUAL;
  return DONE;
}

// The first of several conversions that is not DONE.
#define FIRST(a) do { if (rc == DONE) rc = (a); } while (0)

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
  void *v, *x, *a, *seg, *stream;
  int32_t n_segs, layer;
  Py_buffer p;
  int rc = sort_arguments(names, 9, 7, args, nargs, kwnames, g);
  FIRST(address_of(g[1], &v));
  FIRST(address_of(g[2], &x));
  FIRST(address_of(g[3], &a));
  FIRST(address_of(g[4], &seg));
  FIRST(int32_of(g[5], &n_segs));
  FIRST(int32_of(g[6], &layer));
  FIRST(stream_of(g[7], &stream));
  FIRST(problem_of(g[0], &p));
  if (rc != DONE) return rc < 0 ? NULL : PyObject_Vectorcall(general[SHRINK], args, nargs, kwnames);
  Py_BEGIN_ALLOW_THREADS
  rc = fn_shrink((const sgmv_problem*)p.buf, (float*)v, x, (const void* const*)a, (const int32_t*)seg, n_segs, layer, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[8], "sgmv_shrink");
}

static PyObject* call_expand(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p", "y", "v", "B_ptrs", "seg_starts", "n_segs", "layer_idx", "scale", "stream", "check"};
  PyObject* g[10];
  void *y, *v, *b, *seg, *stream;
  int32_t n_segs, layer;
  float scale;
  Py_buffer p;
  int rc = sort_arguments(names, 10, 8, args, nargs, kwnames, g);
  FIRST(address_of(g[1], &y));
  FIRST(address_of(g[2], &v));
  FIRST(address_of(g[3], &b));
  FIRST(address_of(g[4], &seg));
  FIRST(int32_of(g[5], &n_segs));
  FIRST(int32_of(g[6], &layer));
  FIRST(float_of(g[7], &scale));
  FIRST(stream_of(g[8], &stream));
  FIRST(problem_of(g[0], &p));
  if (rc != DONE) return rc < 0 ? NULL : PyObject_Vectorcall(general[EXPAND], args, nargs, kwnames);
  Py_BEGIN_ALLOW_THREADS
  rc = fn_expand((const sgmv_problem*)p.buf, y, (const float*)v, (const void* const*)b, (const int32_t*)seg, n_segs, layer,
                 scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[9], "sgmv_expand");
}

static PyObject* add_lora(add_lora_fn fn, int which, const char* where, PyObject* const* args, Py_ssize_t nargs,
                          PyObject* kwnames) {
  static const char* const names[] = {"p",      "y",         "x",     "A_ptrs", "B_ptrs", "seg_starts",
                                      "n_segs", "layer_idx", "scale", "stream", "check"};
  PyObject* g[11];
  void *y, *x, *a, *b, *seg, *stream;
  int32_t n_segs, layer;
  float scale;
  Py_buffer p;
  int rc = sort_arguments(names, 11, 9, args, nargs, kwnames, g);
  FIRST(address_of(g[1], &y));
  FIRST(address_of(g[2], &x));
  FIRST(address_of(g[3], &a));
  FIRST(address_of(g[4], &b));
  FIRST(address_of(g[5], &seg));
  FIRST(int32_of(g[6], &n_segs));
  FIRST(int32_of(g[7], &layer));
  FIRST(float_of(g[8], &scale));
  FIRST(stream_of(g[9], &stream));
  FIRST(problem_of(g[0], &p));
  if (rc != DONE) return rc < 0 ? NULL : PyObject_Vectorcall(general[which], args, nargs, kwnames);
  Py_BEGIN_ALLOW_THREADS
  rc = fn((const sgmv_problem*)p.buf, y, x, (const void* const*)a, (const void* const*)b, (const int32_t*)seg, n_segs,
          layer, scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[10], where);
}

static PyObject* call_add_lora(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  return add_lora(fn_add_lora, ADD_LORA, "sgmv_add_lora", args, nargs, kwnames);
}

static PyObject* call_add_lora_static(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  return add_lora(fn_add_lora_static, ADD_LORA_STATIC, "sgmv_add_lora_static", args, nargs, kwnames);
}

// The addresses of a list's or tuple's `n` elements.
// An element's data_ptr() is Python code and may change the very list that is read: the size is looked up
// again and the element kept alive around each one, and what is no longer there counts as NULL.
#define MOST_ADD_ONS 8  // that the library takes; more are left for it to refuse
static int addresses_of(PyObject* seq, Py_ssize_t n, void** out) {
  if (!(PyList_Check(seq) || PyTuple_Check(seq)) || PySequence_Fast_GET_SIZE(seq) != n) return UNUSUAL;
  for (Py_ssize_t i = 0; i < n; ++i) {
    out[i] = NULL;
    if (i >= PySequence_Fast_GET_SIZE(seq)) continue;
    PyObject* element = PySequence_Fast_GET_ITEM(seq, i);
    Py_INCREF(element);
    const int rc = address_of(element, &out[i]);
    Py_DECREF(element);
    if (rc != DONE) return rc;
  }
  return DONE;
}

static PyObject* call_add_lora_multi(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static const char* const names[] = {"p",      "ys",        "xs",    "A_ptrs", "B_ptrs", "seg_starts",
                                      "n_segs", "layer_idx", "scale", "stream", "check"};
  PyObject* g[11];
  void *ys[MOST_ADD_ONS], *xs[MOST_ADD_ONS], *as[MOST_ADD_ONS], *bs[MOST_ADD_ONS], *seg, *stream;
  Py_ssize_t n = 0;
  int32_t n_segs, layer;
  float scale;
  Py_buffer p;
  int rc = sort_arguments(names, 11, 9, args, nargs, kwnames, g);
  if (rc == DONE) {
    n = PyList_Check(g[1]) || PyTuple_Check(g[1]) ? PySequence_Fast_GET_SIZE(g[1]) : MOST_ADD_ONS + 1;
    if (n > MOST_ADD_ONS) rc = UNUSUAL;
  }
  FIRST(addresses_of(g[1], n, ys));
  FIRST(addresses_of(g[2], n, xs));
  FIRST(addresses_of(g[3], n, as));
  FIRST(addresses_of(g[4], n, bs));
  FIRST(address_of(g[5], &seg));
  FIRST(int32_of(g[6], &n_segs));
  FIRST(int32_of(g[7], &layer));
  FIRST(float_of(g[8], &scale));
  FIRST(stream_of(g[9], &stream));
  FIRST(problem_of(g[0], &p));
  if (rc != DONE) return rc < 0 ? NULL : PyObject_Vectorcall(general[ADD_LORA_MULTI], args, nargs, kwnames);
  Py_BEGIN_ALLOW_THREADS
  rc = fn_add_lora_multi((const sgmv_problem*)p.buf, (int32_t)n, ys, (const void* const*)xs, (const void* const* const*)as,
                         (const void* const* const*)bs, (const int32_t*)seg, n_segs, layer, scale, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&p);
  return finish(rc, g[10], "sgmv_add_lora_multi");
}

// bind(problem type, error type, then of sgmv_shrink, sgmv_expand, sgmv_add_lora, sgmv_add_lora_static
// and sgmv_add_lora_multi the addresses and the functions in Python)
static PyObject* call_bind(PyObject* self, PyObject* args) {
  PyObject *problem, *error, *g[5];
  unsigned long long f[5];
  if (!PyArg_ParseTuple(args, "OO(KKKKK)(OOOOO)", &problem, &error, &f[0], &f[1], &f[2], &f[3], &f[4], &g[0], &g[1], &g[2],
                        &g[3], &g[4]))
    return NULL;
  Py_INCREF(problem);
  Py_INCREF(error);
  Py_XSETREF(problem_type, problem);
  Py_XSETREF(error_type, error);
  for (int i = 0; i < 5; ++i) {
    Py_INCREF(g[i]);
    Py_XSETREF(general[i], g[i]);
  }
  fn_shrink = (shrink_fn)(uintptr_t)f[SHRINK];
  fn_expand = (expand_fn)(uintptr_t)f[EXPAND];
  fn_add_lora = (add_lora_fn)(uintptr_t)f[ADD_LORA];
  fn_add_lora_static = (add_lora_fn)(uintptr_t)f[ADD_LORA_STATIC];
  fn_add_lora_multi = (add_lora_multi_fn)(uintptr_t)f[ADD_LORA_MULTI];
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
    {"bind", call_bind, METH_VARARGS, "bind(problem_type, error_type, addresses, functions) -> size of the C struct"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sgmv_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__sgmv_call(void) {
  str_data_ptr = PyUnicode_InternFromString("data_ptr");
  str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!str_data_ptr || !str_cuda_stream) return NULL;
  return PyModule_Create(&module);
}
