/* The call path of the Python binding: one function that turns Python objects into the integer arguments of a C-ABI entry
 * point (include/btc.h) and calls it.
 *
 *   call(address, *arguments) -> status
 *
 * An argument is an int (a number, a size, or an address), None (null), a tensor (its data_ptr()), an object with a buffer
 * (a btc_shape: its address), or a sequence of up to 4 of these (a host array of their addresses).  Every parameter
 * of the entry points is an integer or a pointer, so all of them travel as 64-bit integers.  The interpreter's lock is
 * released around the call.
 *
 * A decode product lasts 5 .. 10 us on the GPU; ctypes took 5 of the 9 us that issuing it took. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#define MAX_ARGS 20
#define MAX_LIST 4

static PyObject* s_data_ptr;

static int to_word(PyObject* o, int64_t* out) {
  if (PyLong_Check(o)) {
    uint64_t v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (uint64_t)-1 && PyErr_Occurred()) return -1;
    *out = (int64_t)v;
    return 0;
  }
  if (o == Py_None) {
    *out = 0;
    return 0;
  }
  if (PyObject_CheckBuffer(o)) {
    if (PyIndex_Check(o)) {               /* an integer of numpy's */
      PyObject* v = PyNumber_Index(o);
      if (!v) return -1;
      *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
      Py_DECREF(v);
      return 0;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return -1;
    *out = (int64_t)(intptr_t)b.buf;      /* (the caller's arguments keep the object alive during the call) */
    PyBuffer_Release(&b);
    return 0;
  }
  PyObject* p = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!p) return -1;
  *out = (int64_t)PyLong_AsUnsignedLongLongMask(p);
  Py_DECREF(p);
  return PyErr_Occurred() ? -1 : 0;
}

typedef int64_t W;
typedef int (*Fn)(W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W);

static int list_words(PyObject* seq, int64_t* out) {
  PyObject** items = PySequence_Fast_ITEMS(seq);
  Py_ssize_t len = PySequence_Fast_GET_SIZE(seq);
  /* a longer list is an error of the entry point, which gets its length as an argument of its own */
  for (Py_ssize_t k = 0; k < len && k < MAX_LIST; ++k)
    if (to_word(items[k], &out[k]) < 0) return -1;
  return 0;
}

static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  (void)self;
  int64_t a[MAX_ARGS] = {0}, list[MAX_ARGS][MAX_LIST] = {{0}};
  if (n < 1 || n - 1 > MAX_ARGS) {
    PyErr_SetString(PyExc_TypeError, "call(address, up to 20 arguments)");
    return NULL;
  }
  uint64_t fn = PyLong_AsUnsignedLongLong(args[0]);
  if (PyErr_Occurred()) return NULL;
  for (Py_ssize_t i = 1; i < n; ++i) {
    PyObject* o = args[i];
    if (PyList_Check(o) || PyTuple_Check(o)) {
      if (list_words(o, list[i - 1]) < 0) return NULL;
      a[i - 1] = (int64_t)(intptr_t)list[i - 1];
    } else if (to_word(o, &a[i - 1]) < 0) {
      /* neither a number nor a tensor nor a buffer: another kind of sequence, or an error */
      if (!PyErr_ExceptionMatches(PyExc_AttributeError) || !PySequence_Check(o)) return NULL;
      PyErr_Clear();
      PyObject* seq = PySequence_Fast(o, "an argument is a number, None, a tensor, a buffer or a sequence of these");
      int rc = seq ? list_words(seq, list[i - 1]) : -1;
      Py_XDECREF(seq);
      if (rc < 0) return NULL;
      a[i - 1] = (int64_t)(intptr_t)list[i - 1];
    }
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  /* surplus arguments are ignored by the callee (they are the caller's to clean up) */
  status = ((Fn)(uintptr_t)fn)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13],
                               a[14], a[15], a[16], a[17], a[18], a[19]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call(address, *arguments) -> status"},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__native(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  if (!s_data_ptr) return NULL;
  return PyModule_Create(&module);
}
