/* Calls of C functions with integer and pointer arguments, for the Python binding.
 *
 * Function(address, arguments, result) is a callable with one character per argument: p a pointer (an int, or None for
 * NULL), q int64, i int32, z size_t; result i or q.  ctypes converts the same arguments through objects of their own
 * (0.5 us for a GEMM's ten; 0.13 us here), which counts where a whole call is a launch of 4 us.
 *
 * Every such argument is passed in one 64-bit register or stack slot by the x86-64 System V convention, of which a
 * callee reads the low half if its parameter is 32 bits wide, and arguments beyond a callee's parameters are not seen: one
 * type of call serves every signature.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>
#include <stdint.h>
#include <string.h>

#if !defined(__x86_64__)
#error "the calls below rely on the x86-64 System V convention"
#endif

enum { MAX_ARGS = 24 };

typedef struct {
  PyObject_HEAD
  vectorcallfunc call;
  uintptr_t address;
  int n;
  char args[MAX_ARGS + 1];
  char result;
} Function;

typedef int64_t (*any_function)(int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                                int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                                int64_t, int64_t, int64_t, int64_t);

static PyObject *argument_error; /* ctypes.ArgumentError, what such calls have always raised, and a TypeError */

/* As ctypes converts: an integer's low bits; None only for a pointer.  at: position of the argument. */
static int convert(PyObject *o, char type, Py_ssize_t at, int64_t *v) {
  if (PyLong_Check(o)) {
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    return 0;
  }
  if (type == 'p' && o == Py_None) {
    *v = 0;
    return 0;
  }
  PyObject *i = PyNumber_Index(o); /* numpy integers and the like */
  if (!i) {
    if (PyErr_ExceptionMatches(PyExc_TypeError))
      PyErr_Format(argument_error, "argument %zd: %s expected instead of %.200s", at + 1,
                   type == 'p' ? "an address or None" : "an integer", Py_TYPE(o)->tp_name);
    return -1;
  }
  *v = (int64_t)PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  return 0;
}

static PyObject *function_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *names) {
  const Function *f = (const Function *)self;
  const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
  if (n != f->n || (names && PyTuple_GET_SIZE(names) != 0)) {
    PyErr_Format(PyExc_TypeError, "%d positional arguments expected, %zd given", f->n, n);
    return NULL;
  }
  int64_t a[MAX_ARGS] = {0};
  for (Py_ssize_t i = 0; i < n; ++i)
    if (convert(args[i], f->args[i], i, &a[i])) return NULL;
  int64_t r;
  Py_BEGIN_ALLOW_THREADS
  r = ((any_function)f->address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13],
                                 a[14], a[15], a[16], a[17], a[18], a[19], a[20], a[21], a[22], a[23]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLongLong(f->result == 'i' ? (int64_t)(int32_t)r : r);
}

static PyObject *function_new(PyTypeObject *type, PyObject *args, PyObject *kwargs) {
  unsigned long long address;
  const char *sig, *result;
  if (kwargs && PyDict_GET_SIZE(kwargs)) {
    PyErr_SetString(PyExc_TypeError, "no keyword arguments");
    return NULL;
  }
  if (!PyArg_ParseTuple(args, "Kss", &address, &sig, &result)) return NULL;
  if (!address || strlen(sig) > MAX_ARGS || strspn(sig, "pqiz") != strlen(sig) || strlen(result) != 1 ||
      !strchr("iq", result[0])) {
    PyErr_SetString(PyExc_ValueError, "not an address and a signature");
    return NULL;
  }
  Function *f = (Function *)type->tp_alloc(type, 0);
  if (!f) return NULL;
  f->call = function_call;
  f->address = (uintptr_t)address;
  f->n = (int)strlen(sig);
  strcpy(f->args, sig);
  f->result = result[0];
  return (PyObject *)f;
}

static PyTypeObject function_type = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "_fastcall.Function",
    .tp_basicsize = sizeof(Function),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(Function, call),
    .tp_call = PyVectorcall_Call,
    .tp_new = function_new,
    .tp_doc = "Function(address, arguments, result): see fastcall.c",
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcall(void) {
  if (PyType_Ready(&function_type) < 0) return NULL;
  if (!argument_error) {
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    PyObject *base = ctypes ? PyObject_GetAttrString(ctypes, "ArgumentError") : NULL;
    PyObject *bases = base ? PyTuple_Pack(2, base, PyExc_TypeError) : NULL;
    if (bases) argument_error = PyErr_NewException("_fastcall.ArgumentError", bases, NULL);
    Py_XDECREF(bases);
    Py_XDECREF(base);
    Py_XDECREF(ctypes);
    if (!argument_error) return NULL;
  }
  PyObject *m = PyModule_Create(&module);
  if (!m) return NULL;
  Py_INCREF(&function_type);
  if (PyModule_AddObject(m, "Function", (PyObject *)&function_type) < 0) {
    Py_DECREF(&function_type);
    Py_DECREF(m);
    return NULL;
  }
  return m;
}
