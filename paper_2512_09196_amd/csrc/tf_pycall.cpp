// tf_variant_run as a Python call, for paper_2512_09196_amd/tf.py: the addresses of tensors and the handle of torch's current
// stream taken in native code. A product of 256^3 takes the GPU 3.0 us; a call through ctypes took 7.6 us, 2.5 of them
// for the Stream object of torch.cuda.current_stream() and 1.5 for frames, c_void_p objects and argument conversion,
// and takes 3.3 here, of which 3.0 are the launch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

namespace {

typedef int32_t (*run_fn)(void*, int32_t, const void*, const void*, const void*, void*, void*, size_t, void*);

run_fn g_run = nullptr;
PyObject* g_slow_stream = nullptr;                      // () -> handle of the current stream
PyObject *g_raw_stream = nullptr, *g_device = nullptr;  // the same as g_raw_stream(g_device()), once the GPU is in use
PyObject *g_data_ptr = nullptr, *g_cuda_stream = nullptr;

bool as_address(PyObject* x, uintptr_t* out) {
  if (!PyLong_Check(x)) {
    PyErr_Format(PyExc_TypeError, "expected an address, got %.100s", Py_TYPE(x)->tp_name);
    return false;
  }
  *out = (uintptr_t)PyLong_AsUnsignedLongLongMask(x);
  return !PyErr_Occurred();
}

// None, an address, or a tensor
bool pointer(PyObject* x, void** out) {
  uintptr_t v = 0;
  if (x == Py_None) {
  } else if (PyLong_Check(x)) {
    if (!as_address(x, &v)) return false;
  } else {
    PyObject* r = PyObject_CallMethodNoArgs(x, g_data_ptr);
    if (!r) return false;
    const bool ok = r == Py_None || as_address(r, &v);      // (no address: null)
    Py_DECREF(r);
    if (!ok) return false;
  }
  *out = (void*)v;
  return true;
}

// None (torch's current stream), a handle, or a stream object
bool stream(PyObject* x, void** out) {
  PyObject* r = nullptr;
  if (x == Py_None) {
    if (g_raw_stream) {
      PyObject* dev = PyObject_CallNoArgs(g_device);
      if (!dev) return false;
      r = PyObject_CallOneArg(g_raw_stream, dev);
      Py_DECREF(dev);
    } else {
      r = PyObject_CallNoArgs(g_slow_stream);
    }
  } else if (PyLong_Check(x)) {
    Py_INCREF(x);
    r = x;
  } else {
    r = PyObject_GetAttr(x, g_cuda_stream);
  }
  if (!r) return false;
  uintptr_t v = 0;
  const bool ok = r == Py_None || as_address(r, &v);        // (no handle: the null stream)
  Py_DECREF(r);
  *out = (void*)v;
  return ok;
}

// run(handle, variant, A, B, bias, Y, workspace, workspace_bytes, stream) -> tf_status
PyObject* run(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 9 || !g_run) {
    PyErr_SetString(PyExc_TypeError, "run() takes nine arguments, after bind()");
    return nullptr;
  }
  uintptr_t handle = 0, variant = 0, bytes = 0;
  void *A, *B, *bias, *Y, *ws, *st;
  if (!as_address(a[0], &handle) || !as_address(a[1], &variant) || !pointer(a[2], &A) || !pointer(a[3], &B) || !pointer(a[4], &bias) ||
      !pointer(a[5], &Y) || !pointer(a[6], &ws) || !as_address(a[7], &bytes) || !stream(a[8], &st))
    return nullptr;
  int32_t r;
  Py_BEGIN_ALLOW_THREADS
  r = g_run((void*)handle, (int32_t)variant, A, B, bias, Y, ws, (size_t)bytes, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(r);
}

// bind(address of tf_variant_run, slow_stream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  uintptr_t f = 0;
  if (n != 2 || !PyCallable_Check(a[1])) {
    PyErr_SetString(PyExc_TypeError, "bind(address, callable)");
    return nullptr;
  }
  if (!as_address(a[0], &f)) return nullptr;
  g_run = (run_fn)f;
  Py_INCREF(a[1]);
  Py_XSETREF(g_slow_stream, a[1]);
  Py_RETURN_NONE;
}

// bind_stream(raw_stream, device), or bind_stream(None, None): back to slow_stream
PyObject* bind_stream(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2) {
    PyErr_SetString(PyExc_TypeError, "bind_stream(raw_stream, device)");
    return nullptr;
  }
  const bool none = a[0] == Py_None || a[1] == Py_None;
  PyObject *raw = none ? nullptr : a[0], *dev = none ? nullptr : a[1];
  Py_XINCREF(raw);
  Py_XINCREF(dev);
  Py_XSETREF(g_device, dev);
  Py_XSETREF(g_raw_stream, raw);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"run", (PyCFunction)(void (*)(void))run, METH_FASTCALL, "tf_variant_run"},
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, "address of tf_variant_run and the slow way to the current stream"},
    {"bind_stream", (PyCFunction)(void (*)(void))bind_stream, METH_FASTCALL, "the fast way to the current stream"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tfcall", "tf_variant_run as a Python call", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tfcall(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_data_ptr || !g_cuda_stream) return nullptr;
  return PyModule_Create(&module);
}
