// CPython binding of the two calls that a denoising loop makes over and over: pab_attention and pab_attention_compute.
//
// Small launches are bound by the host: a reused call, which launches nothing, took 1.75 us from Python, of which the library
// took 0.1: 0.55 for the pointers of three tensors, 0.3 for the stream, 0.45 for ctypes, the rest for the steps in between.
// (With it: a reused call 0.37, an operation of its own 5.8 - 6.2 -> 3.1 - 3.7 with its launch, a run of 60 calls over a tiny model
// 211 - 228 -> 121 - 145, three machines, each without and with it.)
// Here plain torch tensors are looked at through torch's own C++ interface and the library is called directly.  Whatever is not
// a plain dense device tensor or a plain number goes back to the Python code (NotImplemented), which has the same checks and
// raises the errors.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/pab.h"

namespace {

PyObject *py_check, *get_device, *get_raw_stream;   // pab._check; torch's functions for the current device and stream, or NULL

// device address of a plain dense device tensor; false: not one
bool plain_address(PyObject *o, void **p) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) return false;
  *p = t.data_ptr();
  return true;
}

// ... or an address as such (None: 0)
bool address(PyObject *o, void **p) {
  if (plain_address(o, p)) return true;
  if (o == Py_None) *p = nullptr;
  else if (PyLong_CheckExact(o)) *p = PyLong_AsVoidPtr(o);
  else return false;
  return !PyErr_Occurred();
}

bool integer(PyObject *o, int *v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = (int)PyLong_AsLong(o);
  return !PyErr_Occurred();
}

// handle of the stream argument: an address, or None for torch's current stream where a device tensor shows that torch's device
// side is up
bool stream_of(PyObject *o, bool on_device, void **st) {
  if (PyLong_CheckExact(o)) {
    *st = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
  }
  if (o != Py_None || !on_device || !get_raw_stream) return false;
  PyObject *dev = PyObject_CallNoArgs(get_device);
  PyObject *r = dev ? PyObject_CallOneArg(get_raw_stream, dev) : nullptr;
  Py_XDECREF(dev);
  if (!r) return false;
  *st = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

// what the Python code takes over: anything out of the ordinary, of which it raises the errors
PyObject *not_mine() {
  PyErr_Clear();
  Py_RETURN_NOTIMPLEMENTED;
}

// an error status: pab._check raises it
PyObject *failed(int status) {
  PyObject *r = PyObject_CallFunction(py_check, "i", status);
  Py_XDECREF(r);
  if (r) PyErr_SetString(PyExc_RuntimeError, "libpab failed");
  return nullptr;
}

// C++ exceptions end here: a tensor without storage and the like
template <typename F> PyObject *guarded(F f) {
  try {
    return f();
  } catch (const std::exception &) {
    return not_mine();
  }
}

// attention(context address, block, kind, step, q, k, v, stream) -> (decision, address of the slot or None)
PyObject *attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 8) return PyErr_Format(PyExc_TypeError, "attention takes 8 arguments, not %zd", n);
  return guarded([&]() -> PyObject * {
    void *ctx, *q, *k, *v, *st;
    const void *out = nullptr;
    int block, kind, step;
    if (!address(a[0], &ctx) || !integer(a[1], &block) || !integer(a[2], &kind) || !integer(a[3], &step) || !address(a[4], &q) ||
        !address(a[5], &k) || !address(a[6], &v) || !stream_of(a[7], THPVariable_CheckExact(a[4]), &st))
      return not_mine();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = pab_attention(static_cast<pab_ctx *>(ctx), block, kind, step, q, k, v, st, &out);
    Py_END_ALLOW_THREADS
    if (rc < 0) return failed(rc);
    return out ? Py_BuildValue("(iN)", rc, PyLong_FromVoidPtr(const_cast<void *>(out))) : Py_BuildValue("(iO)", rc, Py_None);
  });
}

// attention_compute(kind, q, k, v, out, stream) -> None
PyObject *attention_compute(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 6) return PyErr_Format(PyExc_TypeError, "attention_compute takes 6 arguments, not %zd", n);
  return guarded([&]() -> PyObject * {
    int kind;
    void *p[4], *st;
    if (!integer(a[0], &kind)) return not_mine();
    for (int i = 0; i < 4; ++i)
      if (!plain_address(a[1 + i], &p[i])) return not_mine();
    const at::Tensor &q = THPVariable_Unpack(a[1]), &k = THPVariable_Unpack(a[2]), &v = THPVariable_Unpack(a[3]);
    const auto type = q.scalar_type();
    if ((type != at::kBFloat16 && type != at::kFloat) || k.scalar_type() != type || v.scalar_type() != type || q.dim() != 4) return not_mine();
    const auto s = q.sizes();
    if (k.sizes() != v.sizes()) return not_mine();
    if (kind == PAB_CROSS ? k.dim() != 3 || k.size(1) != s[2] || k.size(2) != s[3] : k.sizes() != s) return not_mine();
    const int64_t L = kind == PAB_CROSS ? k.size(0) : 0;
    for (int64_t x : {s[0], s[1], s[2], s[3], L})
      if (x > 0x7fffffff) return not_mine();
    if (!stream_of(a[5], true, &st)) return not_mine();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = pab_attention_compute(kind, type == at::kBFloat16 ? PAB_BF16 : PAB_F32, (int)s[0], (int)s[1], (int)L, (int)s[2], (int)s[3], p[0],
                               p[1], p[2], p[3], st);
    Py_END_ALLOW_THREADS
    if (rc < 0) return failed(rc);
    Py_RETURN_NONE;
  });
}

// bind(pab._check, torch's current device function, its raw stream function; None where there is none)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 3) return PyErr_Format(PyExc_TypeError, "bind takes 3 arguments, not %zd", n);
  PyObject **slot[3] = {&py_check, &get_device, &get_raw_stream};
  for (int i = 0; i < 3; ++i) {
    PyObject *old = *slot[i];
    *slot[i] = a[i] == Py_None ? nullptr : Py_NewRef(a[i]);
    Py_XDECREF(old);
  }
  if (!get_device) Py_CLEAR(get_raw_stream);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"attention", (PyCFunction)(void (*)(void))attention, METH_FASTCALL, nullptr},
                         {"attention_compute", (PyCFunction)(void (*)(void))attention_compute, METH_FASTCALL, nullptr},
                         {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
