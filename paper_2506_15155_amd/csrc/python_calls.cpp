// The calls that a serving loop makes for every layer of every step, for Python: argument conversion in native code. A wrapper
// of binding.py took 1.3 us to convert its arguments and ctypes another 1.5 to pass them on, beside 2.9 of the call itself;
// here it is 0.6 in all. us a pass that the host bounds: a decode call of four short requests 7.37 -> 5.93, one of a few hundred
// tokens 7.7 -> 6.2.
//
// Only the plain case is handled: the pool an int, ids (and n_new) one-dimensional contiguous numpy arrays of 32-bit integers, device
// buffers None, ints or objects with data_ptr(), the stream None or an int. For anything else, and while torch has not
// initialised the GPU, a function returns None and has done nothing: binding.py then converts the arguments itself.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <numpy/ndarraytypes.h>

#include <cstdint>

namespace {

typedef int (*decode_fn)(void*, const int32_t*, int32_t, const void*, void*, float, void*);
typedef int (*append_decode_fn)(void*, const int32_t*, int32_t, const void*, const void*, const void*, void*, float, void*);
typedef int (*append_fn)(void*, const int32_t*, int32_t, const int32_t*, const void*, const void*, void*);
typedef int (*premap_fn)(void*, const int32_t*, int32_t, uint32_t, int32_t*);

decode_fn decode_of[2];
append_decode_fn append_decode_of;
append_fn append_of;
premap_fn premap_of;
PyTypeObject* ndarray;                      // numpy.ndarray
PyObject *cuda_names, *c_names;             // the namespaces of torch.cuda and torch._C, once torch has been imported
PyObject *s_data_ptr, *s_is_initialized, *s_get_device, *s_get_stream;

enum Got { ERROR = -1, NO = 0, YES = 1 };   // an exception is set; not a plain argument; converted

Got pointer(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = nullptr;
    return YES;
  }
  if (PyLong_CheckExact(o)) {
    *out = (void*)(uintptr_t)PyLong_AsUnsignedLongMask(o);
    return PyErr_Occurred() ? ERROR : YES;
  }
  PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!r) {
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return ERROR;
    PyErr_Clear();
    return NO;
  }
  const Got got = PyLong_CheckExact(r) ? YES : NO;
  if (got) *out = (void*)(uintptr_t)PyLong_AsUnsignedLongMask(r);
  Py_DECREF(r);
  return got;
}

Got numbers(PyObject* o, const int32_t** data, int32_t* n) {
  if (Py_TYPE(o) != ndarray) return NO;
  PyArrayObject* a = (PyArrayObject*)o;
  if (PyArray_NDIM(a) != 1 || PyArray_TYPE(a) != NPY_INT32 || !PyArray_CHKFLAGS(a, NPY_ARRAY_C_CONTIGUOUS | NPY_ARRAY_ALIGNED) ||
      PyArray_DESCR(a)->byteorder == NPY_OPPBYTE)
    return NO;
  const npy_intp size = PyArray_DIM(a, 0);
  if (size < 1 || size > 0x7fffffff) return NO;
  *data = (const int32_t*)PyArray_DATA(a);
  *n = (int32_t)size;
  return YES;
}

Got stream_of(PyObject* o, void** out) {
  if (o != Py_None) return PyLong_CheckExact(o) ? pointer(o, out) : NO;
  // torch's current stream, as binding.py asks for it (looked up each time: these are the names that it uses)
  if (!cuda_names) return NO;
  PyObject *up = PyDict_GetItemWithError(cuda_names, s_is_initialized), *device = PyDict_GetItemWithError(c_names, s_get_device),
           *stream = PyDict_GetItemWithError(c_names, s_get_stream);
  if (!up || !device || !stream) return PyErr_Occurred() ? ERROR : NO;
  PyObject* yes = PyObject_CallNoArgs(up);
  if (!yes) return ERROR;
  const int is_up = PyObject_IsTrue(yes);
  Py_DECREF(yes);
  if (is_up <= 0) return is_up < 0 ? ERROR : NO;
  PyObject* d = PyObject_CallNoArgs(device);
  if (!d) return ERROR;
  PyObject* s = PyObject_CallOneArg(stream, d);
  Py_DECREF(d);
  if (!s) return ERROR;
  const Got got = PyLong_CheckExact(s) ? pointer(s, out) : NO;
  Py_DECREF(s);
  return got;
}

Got number(PyObject* o, float* out) {
  if (!PyFloat_CheckExact(o)) return NO;
  *out = (float)PyFloat_AS_DOUBLE(o);
  return YES;
}

#define TAKE(conversion)                                 \
  do {                                                   \
    const Got got_ = (conversion);                       \
    if (got_ != YES) {                                   \
      if (got_ == ERROR) return nullptr;                 \
      Py_RETURN_NONE;                                    \
    }                                                    \
  } while (0)

// what the arguments of all of these begin with: pool, ids
Got pool_and_ids(PyObject* const* a, void** pool, const int32_t** ids, int32_t* n) {
  if (!PyLong_CheckExact(a[0])) return NO;
  const Got got = pointer(a[0], pool);
  return got == YES ? numbers(a[1], ids, n) : got;
}

bool count(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected", want);
  return false;
}

// (0: ellm_decode_attention, 1: ellm_decode_attention_noalloc; pool, ids, q, out, scale, stream)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (!count(n_args, 7)) return nullptr;
  const decode_fn fn = decode_of[a[0] == Py_True];
  void *pool, *q, *out, *stream;
  const int32_t* ids;
  int32_t n;
  float scale;
  TAKE(pool_and_ids(a + 1, &pool, &ids, &n));
  TAKE(number(a[5], &scale));
  TAKE(stream_of(a[6], &stream));
  TAKE(pointer(a[3], &q));
  TAKE(pointer(a[4], &out));
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(pool, ids, n, q, out, scale, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (pool, ids, k_new, v_new, q, out, scale, stream)
PyObject* append_decode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (!count(n_args, 8)) return nullptr;
  void *pool, *k, *v, *q, *out, *stream;
  const int32_t* ids;
  int32_t n;
  float scale;
  TAKE(pool_and_ids(a, &pool, &ids, &n));
  TAKE(number(a[6], &scale));
  TAKE(stream_of(a[7], &stream));
  TAKE(pointer(a[2], &k));
  TAKE(pointer(a[3], &v));
  TAKE(pointer(a[4], &q));
  TAKE(pointer(a[5], &out));
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = append_decode_of(pool, ids, n, k, v, q, out, scale, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (pool, ids, k_new, v_new, n_new, stream)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (!count(n_args, 6)) return nullptr;
  void *pool, *k, *v, *stream;
  const int32_t *ids, *n_new = nullptr;
  int32_t n, n_n;
  TAKE(pool_and_ids(a, &pool, &ids, &n));
  if (a[4] != Py_None) {
    TAKE(numbers(a[4], &n_new, &n_n));
    if (n_n < n) Py_RETURN_NONE;               // refused by binding.py
  }
  TAKE(stream_of(a[5], &stream));
  TAKE(pointer(a[2], &k));
  TAKE(pointer(a[3], &v));
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = append_of(pool, ids, n, n_new, k, v, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (pool, ids, flags) -> chunks mapped, or the error
PyObject* premap_next(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (!count(n_args, 3)) return nullptr;
  void *pool, *flags;
  const int32_t* ids;
  int32_t n, mapped = 0;
  TAKE(pool_and_ids(a, &pool, &ids, &n));
  if (!PyLong_CheckExact(a[2])) Py_RETURN_NONE;
  TAKE(pointer(a[2], &flags));
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = premap_of(pool, ids, n, (uint32_t)(uintptr_t)flags, &mapped);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc ? rc : mapped);
}

// (numpy.ndarray, addresses of ellm_decode_attention, _noalloc, ellm_kv_append_decode, ellm_kv_append, ellm_kv_premap_next)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject* type;
  unsigned long long f[5];
  if (!PyArg_ParseTuple(args, "OKKKKK", &type, f, f + 1, f + 2, f + 3, f + 4)) return nullptr;
  if (!PyType_Check(type)) {
    PyErr_SetString(PyExc_TypeError, "numpy.ndarray expected");
    return nullptr;
  }
  Py_INCREF(type);
  ndarray = (PyTypeObject*)type;
  decode_of[0] = (decode_fn)f[0];
  decode_of[1] = (decode_fn)f[1];
  append_decode_of = (append_decode_fn)f[2];
  append_of = (append_fn)f[3];
  premap_of = (premap_fn)f[4];
  Py_RETURN_NONE;
}

// (vars(torch.cuda), vars(torch._C))
PyObject* bind_torch(PyObject*, PyObject* args) {
  PyObject *cuda, *c;
  if (!PyArg_ParseTuple(args, "O!O!", &PyDict_Type, &cuda, &PyDict_Type, &c)) return nullptr;
  Py_INCREF(cuda);
  Py_INCREF(c);
  Py_XDECREF(cuda_names);
  Py_XDECREF(c_names);
  cuda_names = cuda;
  c_names = c;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"decode", (PyCFunction)(void (*)(void))decode, METH_FASTCALL, nullptr},
    {"append_decode", (PyCFunction)(void (*)(void))append_decode, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)(void))append, METH_FASTCALL, nullptr},
    {"premap_next", (PyCFunction)(void (*)(void))premap_next, METH_FASTCALL, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {"bind_torch", bind_torch, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_is_initialized = PyUnicode_InternFromString("is_initialized");
  s_get_device = PyUnicode_InternFromString("_cuda_getDevice");
  s_get_stream = PyUnicode_InternFromString("_cuda_getCurrentRawStream");
  if (!s_data_ptr || !s_is_initialized || !s_get_device || !s_get_stream) return nullptr;
  return PyModule_Create(&module);
}
