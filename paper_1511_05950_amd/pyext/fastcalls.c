/* CPython entry points of the calls a training loop makes per gradient and per update.  Same calls and errors as through
 * ctypes; what they save is the argument conversion (a ctypes call with out-parameters costs about a microsecond, these about
 * a tenth), which bounds small networks: at 30-softsync an update of the CIFAR-shaped net takes about 10 us of GPU time and
 * six calls.  Linked against libsasgd.so, which lies next to this module. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/sasgd.h"

static PyObject* error_class;     /* binding.SasgdError(code, message) */
static PyObject* s_data_ptr;      /* "data_ptr" */
static PyObject* s_ctypes;        /* "ctypes" */
static PyObject* s_data;          /* "data" */

static PyObject* raise_code(int code, const char* msg) {
  PyObject* exc = PyObject_CallFunction(error_class, "is", code, msg);
  if (exc) {
    PyErr_SetObject(error_class, exc);
    Py_DECREF(exc);
  }
  return NULL;
}
static PyObject* raise_ctx(sasgd_ctx* ctx, int code) { return raise_code(code, sasgd_last_error(ctx)); }

/* Address of None, an integer, a torch tensor or a numpy array; -1 on error (exception set). */
static int address(PyObject* o, void** out) {
  PyObject* v;
  if (o == Py_None) {
    *out = NULL;
    return 0;
  }
  if (PyLong_Check(o)) {
    *out = PyLong_AsVoidPtr(o);
    return PyErr_Occurred() ? -1 : 0;
  }
  v = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!v) {
    PyObject* c;
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
    PyErr_Clear();
    c = PyObject_GetAttr(o, s_ctypes);
    v = c ? PyObject_GetAttr(c, s_data) : NULL;
    Py_XDECREF(c);
    if (!v) {
      PyErr_SetObject(PyExc_TypeError, (PyObject*)Py_TYPE(o));
      return -1;
    }
  }
  *out = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return PyErr_Occurred() ? -1 : 0;
}

/* Python and numpy integers; a float is refused, as ctypes refuses it. */
static int integer(PyObject* o, long long* out) {
  PyObject* v;
  if (PyLong_Check(o)) {
    *out = PyLong_AsLongLong(o);
    return *out == -1 && PyErr_Occurred() ? -1 : 0;
  }
  v = PyNumber_Index(o);
  if (!v) return -1;
  *out = PyLong_AsLongLong(v);
  Py_DECREF(v);
  return *out == -1 && PyErr_Occurred() ? -1 : 0;
}
static int integer32(PyObject* o, int32_t* out) {
  long long v;
  if (integer(o, &v)) return -1;
  if (v < INT32_MIN || v > INT32_MAX) {
    PyErr_SetString(PyExc_OverflowError, "value does not fit 32 bits");
    return -1;
  }
  *out = (int32_t)v;
  return 0;
}

/* The same with int() applied first: staleness values of any numeric type. */
static int as_integer32(PyObject* o, int32_t* out) {
  PyObject* v;
  int bad;
  if (PyLong_Check(o)) return integer32(o, out);
  v = PyNumber_Long(o);
  if (!v) return -1;
  bad = integer32(v, out);
  Py_DECREF(v);
  return bad;
}

#define NARGS(n) \
  if (nargs != (n)) return PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", (n), nargs)
#define CTX(o)                      \
  void* h;                          \
  sasgd_ctx* ctx;                   \
  if (address((o), &h)) return NULL; \
  ctx = (sasgd_ctx*)h

static PyObject* get_minibatch(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  int32_t learner;
  void *x, *y;
  int rc;
  NARGS(4);
  CTX(a[0]);
  if (integer32(a[1], &learner) || address(a[2], &x) || address(a[3], &y)) return NULL;
  rc = sasgd_getMinibatch(ctx, learner, (const float*)x, (const int32_t*)y);
  if (rc) return raise_ctx(ctx, rc);
  Py_RETURN_NONE;
}

static PyObject* pull_weights(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  int32_t learner, stale;
  int64_t ts = 0;
  int rc;
  NARGS(3);
  CTX(a[0]);
  if (integer32(a[1], &learner) || integer32(a[2], &stale)) return NULL;
  rc = sasgd_pullWeights(ctx, learner, stale, &ts);
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLongLong(ts);
}

static PyObject* push_gradient(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  int32_t learner, tau = 0;
  int rc;
  NARGS(2);
  CTX(a[0]);
  if (integer32(a[1], &learner)) return NULL;
  rc = sasgd_pushGradient(ctx, learner, &tau);
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLong(tau);
}

static PyObject* push_gradient_external(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  void* g;
  long long ts;
  int32_t tau = 0;
  int rc;
  NARGS(3);
  CTX(a[0]);
  if (address(a[1], &g) || integer(a[2], &ts)) return NULL;
  rc = sasgd_pushGradientExternal(ctx, (const float*)g, ts, &tau);
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLong(tau);
}

static PyObject* sum_gradients(PyObject* self, PyObject* h0) {
  int32_t pending = 0;
  int rc;
  CTX(h0);
  rc = sasgd_sumGradients(ctx, &pending);
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLong(pending);
}

static PyObject* apply_update(PyObject* self, PyObject* h0) {
  int64_t ts = 0;
  int rc;
  CTX(h0);
  Py_BEGIN_ALLOW_THREADS            /* calls that may launch kernels leave the interpreter to other threads, as ctypes does */
  rc = sasgd_applyUpdate(ctx, &ts);
  Py_END_ALLOW_THREADS
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLongLong(ts);
}

static PyObject* timestamp(PyObject* self, PyObject* h0) {
  int64_t ts = 0;
  int rc;
  CTX(h0);
  rc = sasgd_timestamp(ctx, &ts);
  if (rc) return raise_ctx(ctx, rc);
  return PyLong_FromLongLong(ts);
}

/* A learner list: at most as many entries as a context can have learners (more is refused by the library's own check of the
 * count, which needs no entry beyond the first). */
#define MOST 64
static PyObject* calc_gradient(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  int32_t ids[MOST];
  Py_ssize_t n, k;
  void* loss;
  PyObject* seq;
  int rc;
  NARGS(3);
  CTX(a[0]);
  if (address(a[2], &loss)) return NULL;
  seq = PySequence_Fast(a[1], "learners must be a sequence");
  if (!seq) return NULL;
  n = PySequence_Fast_GET_SIZE(seq);
  for (k = 0; k < n && k < MOST; k++)
    if (integer32(PySequence_Fast_GET_ITEM(seq, k), &ids[k])) {
      Py_DECREF(seq);
      return NULL;
    }
  Py_DECREF(seq);
  Py_BEGIN_ALLOW_THREADS
  rc = sasgd_calcGradient(ctx, ids, n > MOST ? MOST + 1 : (int32_t)n, (float*)loss);
  Py_END_ALLOW_THREADS
  if (rc) return raise_ctx(ctx, rc);
  Py_RETURN_NONE;
}

/* apply_update_no_alloc(theta_in, theta_out, v, shadow, num_params, grads, staleness, lr_mode, alpha0, momentum, weight_decay,
 * stream) */
static PyObject* apply_update_no_alloc(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  void *tin, *tout, *v, *shadow, *stream;
  long long P;
  int32_t mode, stale[SASGD_NOALLOC_MAX_GRADIENTS];
  const float* grads[SASGD_NOALLOC_MAX_GRADIENTS];
  double alpha0, momentum, decay;
  Py_ssize_t c, k, nst;
  PyObject *gs, *ss;
  char err[256] = "";
  int rc, bad = 0;
  NARGS(12);
  if (address(a[0], &tin) || address(a[1], &tout) || address(a[2], &v) || address(a[3], &shadow) || integer(a[4], &P) ||
      integer32(a[7], &mode) || address(a[11], &stream))
    return NULL;
  alpha0 = PyFloat_AsDouble(a[8]);
  momentum = PyFloat_AsDouble(a[9]);
  decay = PyFloat_AsDouble(a[10]);
  if (PyErr_Occurred()) return NULL;
  gs = PySequence_Fast(a[5], "grads_dev must be a sequence");
  if (!gs) return NULL;
  ss = PySequence_Fast(a[6], "staleness must be a sequence");
  if (!ss) {
    Py_DECREF(gs);
    return NULL;
  }
  c = PySequence_Fast_GET_SIZE(gs);
  nst = PySequence_Fast_GET_SIZE(ss);
  if (nst > (c ? c : 1)) {                  /* one staleness per gradient; missing ones read as 0, as an array of c zeros does */
    PyErr_SetString(PyExc_IndexError, "more staleness values than gradients");
    bad = 1;
  }
  for (k = 0; !bad && k < c && k < SASGD_NOALLOC_MAX_GRADIENTS; k++) {
    void* g;
    stale[k] = 0;
    bad = address(PySequence_Fast_GET_ITEM(gs, k), &g) || (k < nst && as_integer32(PySequence_Fast_GET_ITEM(ss, k), &stale[k]));
    grads[k] = (const float*)g;
  }
  Py_DECREF(gs);
  Py_DECREF(ss);
  if (bad) return NULL;
  Py_BEGIN_ALLOW_THREADS
  rc = sasgd_applyUpdateNoAlloc((const float*)tin, (float*)tout, (float*)v, (uint16_t*)shadow, P,
                                c > SASGD_NOALLOC_MAX_GRADIENTS ? SASGD_NOALLOC_MAX_GRADIENTS + 1 : (int32_t)c, grads, stale, mode, (float)alpha0,
                                (float)momentum, (float)decay, stream, err, sizeof(err));
  Py_END_ALLOW_THREADS
  if (rc) return raise_code(rc, err);
  return PyLong_FromLong(rc);
}

static PyObject* set_error_class(PyObject* self, PyObject* cls) {
  Py_INCREF(cls);
  Py_XDECREF(error_class);
  error_class = cls;
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {FAST(get_minibatch),
                                FAST(pull_weights),
                                FAST(push_gradient),
                                FAST(push_gradient_external),
                                FAST(calc_gradient),
                                FAST(apply_update_no_alloc),
                                {"sum_gradients", sum_gradients, METH_O, NULL},
                                {"apply_update", apply_update, METH_O, NULL},
                                {"timestamp", timestamp, METH_O, NULL},
                                {"set_error_class", set_error_class, METH_O, NULL},
                                {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcalls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcalls(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_ctypes = PyUnicode_InternFromString("ctypes");
  s_data = PyUnicode_InternFromString("data");
  if (!s_data_ptr || !s_ctypes || !s_data) return NULL;
  Py_INCREF(PyExc_RuntimeError);
  error_class = PyExc_RuntimeError;
  return PyModule_Create(&module);
}
