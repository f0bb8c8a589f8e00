/* Calls of the library's C entries from Python with less on the way than ctypes has: call(address, descriptor, ...) passes a
 * descriptor (any object with a buffer) by its address, a tensor by its data_ptr(), None as 0 and integers as they are, and
 * returns the status.  A decode step's projection is a call whose kernel takes 4 us: through ctypes and torch's stream
 * objects it was 9.0 us of the host's time, 4.2 of them the C entry's own (4096 x 4096, 3-bit, one vector). */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#define MOST 8
typedef int (*entry_t)(int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t);

static PyObject* data_ptr;                     /* the name */

/* The entries take integers and pointers only, at most MOST of them: in the x86-64 calling convention each is a register or
 * an 8-byte stack slot whatever its width, and those that an entry has no parameter for are not looked at. */
static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  int64_t v[MOST] = {0};
  Py_buffer descriptor;
  (void)self;
  if (n < 2 || n > MOST + 1) {
    PyErr_SetString(PyExc_TypeError, "call(address, descriptor, ...) takes up to 8 arguments behind the address");
    return NULL;
  }
  const unsigned long long address = PyLong_AsUnsignedLongLong(args[0]);
  if (address == (unsigned long long)-1 && PyErr_Occurred()) return NULL;
  if (PyObject_GetBuffer(args[1], &descriptor, PyBUF_SIMPLE) != 0) return NULL;
  v[0] = (int64_t)(intptr_t)descriptor.buf;
  PyObject* result = NULL;
  for (Py_ssize_t i = 2; i < n; ++i) {
    PyObject* a = args[i];
    if (a == Py_None) continue;
    PyObject* number = NULL;
    if (PyLong_Check(a)) {
      number = PyNumber_Index(a);
    } else {                                   /* a tensor is its address, also where it could be an index */
      number = PyObject_CallMethodNoArgs(a, data_ptr);
      if (number == NULL && PyErr_ExceptionMatches(PyExc_AttributeError)) {
        PyErr_Clear();
        number = PyNumber_Index(a);
      }
    }
    if (number == NULL) goto done;
    /* addresses are unsigned, sizes and dtypes are not: the low 64 bits of either */
    v[i - 1] = (int64_t)PyLong_AsUnsignedLongLongMask(number);
    Py_DECREF(number);
    if (v[i - 1] == -1 && PyErr_Occurred()) goto done;
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = ((entry_t)(uintptr_t)address)(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
  Py_END_ALLOW_THREADS
  result = PyLong_FromLong(status);
done:
  PyBuffer_Release(&descriptor);
  return result;
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__calls(void) {
  data_ptr = PyUnicode_InternFromString("data_ptr");
  return data_ptr == NULL ? NULL : PyModule_Create(&module);
}
