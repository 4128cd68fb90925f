// The two calls of a decode step from Python without ctypes: addresses out of the argument objects, the current stream's
// handle, the library's function, its status back.  Everything else stays with the ctypes binding (qaq.py), whose checks and
// messages these are.
//
// A short step's kernels take about as long as its calls take the host.  Through ctypes and a Python function per argument one
// attention call of 8 heads x 512 tokens was 8.5 us, 24 steps of a small model 395; so 7.4 and 377.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*attention_fn)(void*, const void*, const void*, const void*, void*, int32_t, float*, void*);
typedef int (*update_fn)(void*, const float*, const void*, const void*, void*, void*, int32_t, uint8_t*, uint8_t*, void*);

static PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_dev_ptr, *s_dtype;      // attribute names
static PyObject *host_buffer, *float32, *get_device, *raw_stream, *any_stream;          // see setup()

// Address of a device tensor, or the device's address of a page-locked buffer; None: NULL.  -1 and an exception where it is neither.
static int address(PyObject* t, void** out) {
  *out = NULL;
  if (t == Py_None) return 0;
  PyObject* at;
  if (PyObject_TypeCheck(t, (PyTypeObject*)host_buffer)) {
    at = PyObject_GetAttr(t, s_dev_ptr);
  } else {
    PyObject* x = PyObject_GetAttr(t, s_is_cuda);
    int ok = x ? PyObject_IsTrue(x) : -1;
    Py_XDECREF(x);
    if (ok > 0) {
      x = PyObject_CallMethodNoArgs(t, s_is_contiguous);
      ok = x ? PyObject_IsTrue(x) : -1;
      Py_XDECREF(x);
    }
    if (ok < 0) return -1;
    if (!ok) {
      PyErr_SetString(PyExc_AssertionError, "device tensors must be contiguous CUDA tensors");
      return -1;
    }
    at = PyObject_CallMethodNoArgs(t, s_data_ptr);
  }
  if (!at) return -1;
  if (at != Py_None) *out = PyLong_AsVoidPtr(at);
  Py_DECREF(at);
  return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

// The current stream of the current device: by torch's own lookups (asking for the device has torch's checks: a GPU, no fork
// since it was first used), or, where it has them not, by the function that qaq.py has for that.
static int stream(void** out) {
  PyObject* s;
  if (raw_stream != Py_None) {
    PyObject* dev = PyObject_CallNoArgs(get_device);
    if (!dev) return -1;
    s = PyObject_CallOneArg(raw_stream, dev);
    Py_DECREF(dev);
  } else {
    s = PyObject_CallNoArgs(any_stream);
  }
  if (!s) return -1;
  *out = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

static int pointer(PyObject* o, void** out) {
  *out = PyLong_AsVoidPtr(o);
  return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

static PyObject* wrong_count(const char* name) {
  PyErr_Format(PyExc_TypeError, "%s: wrong number of arguments", name);
  return NULL;
}

// attention(function, cache, q, k_new, v_new, out, scores) -> status
static PyObject* attention(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  (void)self;
  void *fn, *cache, *p[5], *s;
  if (n != 7) return wrong_count("attention");
  if (!float32) { PyErr_SetString(PyExc_RuntimeError, "setup() has not been called"); return NULL; }
  if (pointer(a[0], &fn) || pointer(a[1], &cache)) return NULL;
  for (int i = 0; i < 5; ++i)
    if (address(a[2 + i], &p[i])) return NULL;
  PyObject* dt = PyObject_GetAttr(a[5], s_dtype);
  if (!dt) return NULL;
  const int is_fp32 = dt == float32;
  Py_DECREF(dt);
  if (stream(&s)) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = ((attention_fn)fn)(cache, p[0], p[1], p[2], p[3], is_fp32, (float*)p[4], s);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// update(function, cache, scores, k_new, v_new, k_orig, v_orig, orig_tokens, k_bits, v_bits) -> status
static PyObject* update(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  (void)self;
  void *fn, *cache, *p[5], *bits[2], *s;
  if (n != 10) return wrong_count("update");
  if (!float32) { PyErr_SetString(PyExc_RuntimeError, "setup() has not been called"); return NULL; }
  if (pointer(a[0], &fn) || pointer(a[1], &cache)) return NULL;
  for (int i = 0; i < 5; ++i)
    if (address(a[2 + i], &p[i])) return NULL;
  const long tokens = PyLong_AsLong(a[7]);
  if (tokens == -1 && PyErr_Occurred()) return NULL;
  for (int i = 0; i < 2; ++i)
    if (address(a[8 + i], &bits[i])) return NULL;
  if (stream(&s)) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = ((update_fn)fn)(cache, (const float*)p[0], p[1], p[2], p[3], p[4], (int32_t)tokens, (uint8_t*)bits[0], (uint8_t*)bits[1], s);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// setup(HostBuffer, torch.float32, device lookup or None, stream lookup or None, stream function): once, before the others
static PyObject* setup(PyObject* self, PyObject* args) {
  (void)self;
  PyObject* x[5];
  if (!PyArg_ParseTuple(args, "O!OOOO", &PyType_Type, &x[0], &x[1], &x[2], &x[3], &x[4])) return NULL;
  PyObject** const to[5] = {&host_buffer, &float32, &get_device, &raw_stream, &any_stream};
  for (int i = 0; i < 5; ++i) {
    PyObject* old = *to[i];
    Py_INCREF(x[i]);
    *to[i] = x[i];
    Py_XDECREF(old);
  }
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"attention", (PyCFunction)(void (*)(void))attention, METH_FASTCALL, NULL},
    {"update", (PyCFunction)(void (*)(void))update, METH_FASTCALL, NULL},
    {"setup", setup, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qaq_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__qaq_call(void) {
  struct { PyObject** to; const char* text; } names[] = {
      {&s_is_cuda, "is_cuda"}, {&s_is_contiguous, "is_contiguous"}, {&s_data_ptr, "data_ptr"}, {&s_dev_ptr, "dev_ptr"}, {&s_dtype, "dtype"}};
  for (unsigned i = 0; i < sizeof(names) / sizeof(names[0]); ++i)
    if (!(*names[i].to = PyUnicode_InternFromString(names[i].text))) return NULL;
  return PyModule_Create(&module);
}
