/* _calls: the entry points of libgnmr that a training loop makes every step,
 * called from Python without ctypes.
 *
 * Argument marshalling only, with the conversions of the ctypes binding: a
 * pointer is data_ptr() of what has one, else int(); a stream is cuda_stream of
 * what has one, else int(), None the null stream; int() and float() elsewhere,
 * integers cut to the width of the C argument.  Every function returns the
 * status of the C call, which runs without the interpreter lock.
 *
 * What it is for: the small calls, whose kernels are shorter than their
 * marshalling was, and long lists.  Host time of a call without the C entry
 * point, ctypes with its Python code and here: one actuated matrix 2.2 and
 * 0.65 us, 28 weight-gradient problems 45 and 9 us, 70 segment pointers 12.6
 * and 1.0 us, 12,000 of them 1,550 and 110 us; the kernels beside them take
 * 3.7, 33, 62 and about 650 us.
 *
 * The addresses come from the library that the ctypes binding has loaded, so
 * both always speak to the same build. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <stdlib.h>

#include "gnmr.h"

#define ENTRIES(X)                                                             \
  X(gnmr_step) X(gnmr_step_from_norms) X(gnmr_step_from_partials) X(gnmr_sumsq) \
  X(gnmr_actuate) X(gnmr_actuate_matrix) X(gnmr_wgrad_sumsq) X(gnmr_wgrad_sumsq_batched)
#define DECLARE(f) static __typeof__(&f) p_##f;
ENTRIES(DECLARE)

static PyObject *s_data_ptr, *s_cuda_stream, *s_value;

/* Lists up to this length are marshalled on the stack. */
enum { kOnStack = 256 };

/* -- conversions: 0, or -1 with an exception set ------------------------------ */

static int as_u64(PyObject* o, uint64_t* v) {
  if (PyLong_CheckExact(o)) {
    *v = PyLong_AsUnsignedLongLongMask(o);
    return *v == UINT64_MAX && PyErr_Occurred() ? -1 : 0;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) return -1;
  *v = PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return *v == UINT64_MAX && PyErr_Occurred() ? -1 : 0;
}

static int as_i64(PyObject* o, int64_t* v) { return as_u64(o, (uint64_t*)v); }

static int as_i32(PyObject* o, int32_t* v) {
  uint64_t u;
  if (as_u64(o, &u)) return -1;
  *v = (int32_t)(uint32_t)u;
  return 0;
}

static int as_f64(PyObject* o, double* v) {
  if (PyFloat_CheckExact(o)) {
    *v = PyFloat_AS_DOUBLE(o);
    return 0;
  }
  PyObject* n = PyNumber_Float(o);
  if (!n) return -1;
  *v = PyFloat_AS_DOUBLE(n);
  Py_DECREF(n);
  return 0;
}

/* What ctypes takes for a pointer: an int, or None for a null one. */
static int as_word(PyObject* o, uint64_t* v) {
  *v = 0;
  if (o == Py_None) return 0;
  if (PyLong_Check(o)) return as_u64(o, v);
  PyErr_Format(PyExc_TypeError, "%.100s in place of an address", Py_TYPE(o)->tp_name);
  return -1;
}

static int as_ptr(PyObject* o, void** p) {
  uint64_t u;
  if (!PyLong_CheckExact(o)) {
    PyObject* n = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (n) {
      const int bad = as_word(n, &u);
      Py_DECREF(n);
      *p = (void*)(uintptr_t)u;
      return bad;
    }
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
    /* an AttributeError from inside data_ptr() is the caller's */
    PyObject *t, *v, *tb;
    PyErr_Fetch(&t, &v, &tb);
    if (PyObject_HasAttr(o, s_data_ptr)) {
      PyErr_Restore(t, v, tb);
      return -1;
    }
    Py_XDECREF(t);
    Py_XDECREF(v);
    Py_XDECREF(tb);
  }
  if (as_u64(o, &u)) return -1;
  *p = (void*)(uintptr_t)u;
  return 0;
}

static int as_stream(PyObject* o, void** s) {
  uint64_t u = 0;
  if (o != Py_None && !PyLong_CheckExact(o)) {
    PyObject* n = PyObject_GetAttr(o, s_cuda_stream);
    if (!n) {
      if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
      PyErr_Clear();
      if (as_u64(o, &u)) return -1;
    } else {
      int bad = as_u64(n, &u);
      Py_DECREF(n);
      if (bad) return -1;
    }
  } else if (o != Py_None && as_u64(o, &u)) {
    return -1;
  }
  *s = (void*)(uintptr_t)u;
  return 0;
}

/* A context: None, an int or a ctypes.c_void_p. */
static int as_handle(PyObject* o, void** h) {
  uint64_t u;
  int bad;
  if (o == Py_None || PyLong_Check(o)) {
    bad = as_word(o, &u);
  } else {
    PyObject* n = PyObject_GetAttr(o, s_value);
    if (!n) return -1;
    bad = as_word(n, &u);
    Py_DECREF(n);
  }
  *h = (void*)(uintptr_t)u;
  return bad;
}

/* The pointers of an iterable in `stack` or, past kOnStack, in new memory;
 * NULL with an exception set on failure.  An empty one gives one null pointer. */
static void** as_pointers(PyObject* seq, void** stack) {
  PyObject* t = PySequence_Tuple(seq); /* own references: data_ptr() may run any code */
  if (!t) return NULL;
  const Py_ssize_t n = PyTuple_GET_SIZE(t);
  void** out = stack;
  if (n > kOnStack && !(out = malloc((size_t)n * sizeof *out))) {
    Py_DECREF(t);
    PyErr_NoMemory();
    return NULL;
  }
  if (n == 0) out[0] = NULL;
  for (Py_ssize_t i = 0; i < n; ++i)
    if (as_ptr(PyTuple_GET_ITEM(t, i), out + i)) {
      if (out != stack) free(out);
      Py_DECREF(t);
      return NULL;
    }
  Py_DECREF(t);
  return out;
}

/* (dy, x, dw, tokens, out_features, in_features[, accumulate]) */
static int as_problem(PyObject* o, gnmr_wgrad_problem* p) {
  PyObject* t = NULL;
  int64_t tokens;
  int bad = -1;
  p->accumulate = 0;
  p->reserved = 0;
  if (PyTuple_CheckExact(o) || PyList_CheckExact(o)) {
    t = PySequence_Tuple(o);
  } else { /* what takes p[:6], len(p) and p[6] */
    PyObject* head = PySequence_GetSlice(o, 0, 6);
    if (!head) return -1;
    t = PySequence_Tuple(head);
    Py_DECREF(head);
    const Py_ssize_t len = t ? PyObject_Size(o) : -1;
    if (len < 0) goto done;
    if (len > 6) {
      PyObject* a = PySequence_GetItem(o, 6);
      if (!a) goto done;
      const int no = as_i32(a, &p->accumulate);
      Py_DECREF(a);
      if (no) goto done;
    }
  }
  if (!t) return -1;
  if (PyTuple_GET_SIZE(t) < 6) {
    PyErr_Format(PyExc_ValueError, "not enough values to unpack (expected 6, got %zd)",
                 PyTuple_GET_SIZE(t));
    goto done;
  }
  if (as_ptr(PyTuple_GET_ITEM(t, 0), (void**)&p->dy) ||
      as_ptr(PyTuple_GET_ITEM(t, 1), (void**)&p->x) || as_ptr(PyTuple_GET_ITEM(t, 2), &p->dw) ||
      as_i64(PyTuple_GET_ITEM(t, 3), &tokens) ||
      as_i32(PyTuple_GET_ITEM(t, 4), &p->out_features) ||
      as_i32(PyTuple_GET_ITEM(t, 5), &p->in_features) ||
      (PyTuple_GET_SIZE(t) > 6 && as_i32(PyTuple_GET_ITEM(t, 6), &p->accumulate)))
    goto done;
  p->tokens = tokens;
  bad = 0;
done:
  Py_XDECREF(t);
  return bad;
}

/* -- calls ---------------------------------------------------------------------- */

static int arity(Py_ssize_t got, Py_ssize_t want) {
  if (got == want && p_gnmr_step) return 0;
  if (got != want)
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", got, want);
  else
    PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
  return -1;
}

#define CALL(expr)              \
  int status;                   \
  Py_BEGIN_ALLOW_THREADS        \
  status = (int)(expr);         \
  Py_END_ALLOW_THREADS

static PyObject* step(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *stream, *stack[kOnStack], **ptrs = NULL;
  double alpha, beta;
  if (arity(n, 5) || as_handle(a[0], &ctx) || as_f64(a[1], &alpha) || as_f64(a[2], &beta) ||
      as_stream(a[4], &stream) || (a[3] != Py_None && !(ptrs = as_pointers(a[3], stack))))
    return NULL;
  CALL(p_gnmr_step(ctx, alpha, beta, (const void* const*)ptrs, stream))
  if (ptrs && ptrs != stack) free(ptrs);
  return PyLong_FromLong(status);
}

static PyObject* sumsq(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *stream, *out, *stack[kOnStack], **ptrs = NULL;
  if (arity(n, 4) || as_handle(a[0], &ctx) || as_ptr(a[2], &out) || as_stream(a[3], &stream) ||
      (a[1] != Py_None && !(ptrs = as_pointers(a[1], stack))))
    return NULL;
  CALL(p_gnmr_sumsq(ctx, (const void* const*)ptrs, out, stream))
  if (ptrs && ptrs != stack) free(ptrs);
  return PyLong_FromLong(status);
}

static PyObject* step_from_norms(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *norm, *stream;
  double alpha, beta;
  if (arity(n, 5) || as_handle(a[0], &ctx) || as_ptr(a[1], &norm) || as_f64(a[2], &alpha) ||
      as_f64(a[3], &beta) || as_stream(a[4], &stream))
    return NULL;
  CALL(p_gnmr_step_from_norms(ctx, norm, alpha, beta, stream))
  return PyLong_FromLong(status);
}

static PyObject* step_from_partials(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *part, *stream;
  double alpha, beta;
  if (arity(n, 5) || as_handle(a[0], &ctx) || as_ptr(a[1], &part) || as_f64(a[2], &alpha) ||
      as_f64(a[3], &beta) || as_stream(a[4], &stream))
    return NULL;
  CALL(p_gnmr_step_from_partials(ctx, part, alpha, beta, stream))
  return PyLong_FromLong(status);
}

static PyObject* actuate(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *act, *mask, *stream;
  int32_t low, rec;
  if (arity(n, 5) || as_handle(a[0], &act) || as_ptr(a[1], &mask) || as_i32(a[2], &low) ||
      as_i32(a[3], &rec) || as_stream(a[4], &stream))
    return NULL;
  CALL(p_gnmr_actuate(act, mask, low, rec, stream))
  return PyLong_FromLong(status);
}

static PyObject* actuate_matrix(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *x, *out, *mask, *stream;
  int64_t rows;
  int32_t cols, unit, low, rec;
  if (arity(n, 9) || as_ptr(a[0], &x) || as_ptr(a[1], &out) || as_i64(a[2], &rows) ||
      as_i32(a[3], &cols) || as_ptr(a[4], &mask) || as_i32(a[5], &unit) || as_i32(a[6], &low) ||
      as_i32(a[7], &rec) || as_stream(a[8], &stream))
    return NULL;
  CALL(p_gnmr_actuate_matrix(x, out, rows, cols, mask, unit, low, rec, stream))
  return PyLong_FromLong(status);
}

static PyObject* wgrad_sumsq(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *dy, *x, *dw, *sums, *stream;
  int64_t tokens;
  int32_t outf, inf;
  if (arity(n, 8) || as_ptr(a[0], &dy) || as_ptr(a[1], &x) || as_ptr(a[2], &dw) ||
      as_i64(a[3], &tokens) || as_i32(a[4], &outf) || as_i32(a[5], &inf) || as_ptr(a[6], &sums) ||
      as_stream(a[7], &stream))
    return NULL;
  CALL(p_gnmr_wgrad_sumsq(dy, x, dw, tokens, outf, inf, sums, stream))
  return PyLong_FromLong(status);
}

static PyObject* wgrad_sumsq_batched(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  void *sums, *stream;
  if (arity(n, 3)) return NULL;
  PyObject* t = PySequence_Tuple(a[0]);
  if (!t) return NULL;
  const Py_ssize_t count = PyTuple_GET_SIZE(t);
  gnmr_wgrad_problem* ps = malloc((size_t)(count ? count : 1) * sizeof *ps);
  if (!ps) {
    Py_DECREF(t);
    return PyErr_NoMemory();
  }
  int bad = 0;
  for (Py_ssize_t i = 0; i < count && !bad; ++i) bad = as_problem(PyTuple_GET_ITEM(t, i), ps + i);
  Py_DECREF(t);
  if (bad || as_ptr(a[1], &sums) || as_stream(a[2], &stream)) {
    free(ps);
    return NULL;
  }
  CALL(p_gnmr_wgrad_sumsq_batched(ps, (int32_t)count, sums, stream))
  free(ps);
  return PyLong_FromLong(status);
}

/* bind({name: address}): where the entry points are */
static PyObject* bind(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  if (n != 1 || !PyDict_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "bind() takes a dict of addresses");
    return NULL;
  }
#define ADDRESS(f)                                                        \
  uint64_t u_##f;                                                         \
  {                                                                       \
    PyObject* v = PyDict_GetItemString(a[0], #f);                         \
    if (!v) {                                                             \
      PyErr_SetString(PyExc_KeyError, #f);                                \
      return NULL;                                                        \
    }                                                                     \
    if (as_u64(v, &u_##f)) return NULL;                                   \
  }
  ENTRIES(ADDRESS)
#define STORE(f) p_##f = (__typeof__(p_##f))(uintptr_t)u_##f;
  ENTRIES(STORE)
  Py_RETURN_NONE;
}

#define METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, NULL}
static PyMethodDef kMethods[] = {METHOD(bind),
                                 METHOD(step),
                                 METHOD(sumsq),
                                 METHOD(step_from_norms),
                                 METHOD(step_from_partials),
                                 METHOD(actuate),
                                 METHOD(actuate_matrix),
                                 METHOD(wgrad_sumsq),
                                 METHOD(wgrad_sumsq_batched),
                                 {NULL, NULL, 0, NULL}};
static struct PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, kMethods,
                                     NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void) {
  if (!(s_data_ptr = PyUnicode_InternFromString("data_ptr")) ||
      !(s_cuda_stream = PyUnicode_InternFromString("cuda_stream")) ||
      !(s_value = PyUnicode_InternFromString("value")))
    return NULL;
  return PyModule_Create(&kModule);
}
