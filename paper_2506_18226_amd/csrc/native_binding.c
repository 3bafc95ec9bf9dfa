/* CPython side of binding.py: turns the arguments of the hot entry points into one C call.
 *
 * A decode step of a small batch is bound by what the host does, and a launch itself takes 2.4 us of it.  Marshalled by ctypes
 * and Python code attend_layer took 6.1 us a call and an adsa_step of three launches 11.0; through this module 4.2 and 9.7.
 *
 * A pointer argument is None, an integer, an object with data_ptr() (a torch tensor), or one of these with a byte offset; nothing
 * is kept from one call for the next. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "adsa.h"

static PyObject *s_data_ptr, *s_numel, *s_element_size, *params_type;

/* device address of x: NULL, the integer itself, x.data_ptr(), or for (x, bytes) that many further on (NULL stays NULL); -1 with an exception set */
static int as_pointer(PyObject* x, void** out) {
  if (x == Py_None) { *out = NULL; return 0; }
  if (PyTuple_CheckExact(x) && PyTuple_GET_SIZE(x) == 2) {
    const Py_ssize_t off = PyLong_AsSsize_t(PyTuple_GET_ITEM(x, 1));
    if (PyErr_Occurred() || PyTuple_CheckExact(PyTuple_GET_ITEM(x, 0)) || as_pointer(PyTuple_GET_ITEM(x, 0), out) < 0) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "(pointer, bytes) expected");
      return -1;
    }
    if (*out) *out = (char*)*out + off;
    return 0;
  }
  if (PyLong_Check(x)) {
    *out = PyLong_AsVoidPtr(x);
    return PyErr_Occurred() ? -1 : 0;
  }
  PyObject* p = PyObject_CallMethodNoArgs(x, s_data_ptr);
  if (!p) return -1;
  *out = PyLong_AsVoidPtr(p);
  Py_DECREF(p);
  return PyErr_Occurred() ? -1 : 0;
}

static int as_bytes(PyObject* x, size_t* out) {
  if (x == Py_None) { *out = 0; return 0; }
  PyObject *n = PyObject_CallMethodNoArgs(x, s_numel), *e = n ? PyObject_CallMethodNoArgs(x, s_element_size) : NULL;
  const int ok = n && e;
  if (ok) *out = PyLong_AsSize_t(n) * PyLong_AsSize_t(e);
  Py_XDECREF(n);
  Py_XDECREF(e);
  return ok && !PyErr_Occurred() ? 0 : -1;
}

typedef int (*fn_select)(const void*, void*, void*, void*, uint32_t, void*, size_t, void*);
typedef int (*fn_attend)(const void*, void*, const void*, const void*, const void*, const void*, const void*, void*, void*, uint32_t, void*, size_t, void*);
typedef int (*fn_compact)(const void*, void*, void*, uint32_t, void*, size_t, void*);
typedef int (*fn_step)(const void*, void*, const void*, const void*, const void*, void*, void*, void*, void*, void*, uint32_t, void*, size_t, void*);
typedef int (*fn_step_static)(const void*, void*, const void*, const void*, const void*, void*, void*, void*, void*, void*, uint32_t, void*);

enum { SELECT = 3, ATTEND = 8, COMPACT = 2, STEP = 9 };         /* pointer arguments of the entry points, seqs first */

/* a: address of the C function, params, flags, stream, workspace (has_ws), pointers...  The number of pointers says which entry
 * point it is; adsa_step_static, which has as many as adsa_step, is the one without a workspace. */
static PyObject* call_c(PyObject* const* a, Py_ssize_t n, int has_ws) {
  void *fn, *p[STEP], *ws = NULL, *stream;
  size_t ws_bytes = 0;
  const Py_ssize_t first = has_ws ? 5 : 4, np = n - first;
  if (np != STEP && (!has_ws || (np != SELECT && np != ATTEND && np != COMPACT))) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return NULL;
  }
  if (as_pointer(a[0], &fn) < 0) return NULL;
  const unsigned long flags = PyLong_AsUnsignedLongMask(a[2]);
  if (PyErr_Occurred()) return NULL;
  if (as_pointer(a[3], &stream) < 0) return NULL;
  if (has_ws && (as_pointer(a[4], &ws) < 0 || as_bytes(a[4], &ws_bytes) < 0)) return NULL;
  for (Py_ssize_t i = 0; i < np; ++i)
    if (as_pointer(a[first + i], &p[i]) < 0) return NULL;
  Py_buffer params;
  const int typed = params_type ? PyObject_IsInstance(a[1], params_type) : 0;
  if (typed < 0) return NULL;
  if (!typed) {
    PyErr_SetString(PyExc_TypeError, "params: AdsaParams expected");
    return NULL;
  }
  if (PyObject_GetBuffer(a[1], &params, PyBUF_SIMPLE) < 0) return NULL;
  if (params.len < (Py_ssize_t)sizeof(adsa_params)) {
    PyBuffer_Release(&params);
    PyErr_SetString(PyExc_TypeError, "params: too small");
    return NULL;
  }
  const void* const pp = params.buf;
  const uint32_t f = (uint32_t)flags;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  if (np == ATTEND) rc = ((fn_attend)fn)(pp, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], f, ws, ws_bytes, stream);
  else if (np == SELECT) rc = ((fn_select)fn)(pp, p[0], p[1], p[2], f, ws, ws_bytes, stream);
  else if (np == COMPACT) rc = ((fn_compact)fn)(pp, p[0], p[1], f, ws, ws_bytes, stream);
  else if (has_ws) rc = ((fn_step)fn)(pp, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], f, ws, ws_bytes, stream);
  else rc = ((fn_step_static)fn)(pp, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], f, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&params);
  return PyLong_FromLong(rc);
}

static PyObject* call_entry(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  (void)self;
  return call_c(a, n, 1);
}

static PyObject* call_static(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  (void)self;
  return call_c(a, n, 0);
}

/* the ctypes mirror of adsa_params that the calls take */
static PyObject* set_params_type(PyObject* self, PyObject* type) {
  (void)self;
  Py_INCREF(type);
  Py_XSETREF(params_type, type);
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"set_params_type", set_params_type, METH_O, "The type of the calls' params."},
                                {"call", (PyCFunction)(void (*)(void))call_entry, METH_FASTCALL, "One C call."},
                                {"call_static", (PyCFunction)(void (*)(void))call_static, METH_FASTCALL, "One call of adsa_step_static."}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_adsa_native", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__adsa_native(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  return s_data_ptr && s_numel && s_element_size ? PyModule_Create(&module) : NULL;
}
