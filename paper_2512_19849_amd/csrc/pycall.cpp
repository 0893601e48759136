// The calls of a step from Python: arguments straight from the tensors to the C ABI (include/ep.h).  Marshalling through
// ctypes costs 1.2 us and more a call (ep_combine of no tokens; 0.2 here), nearly as much as the launch behind it, and steps
// of few tokens are bound by the calls of the host.  What is not one of the plain argument kinds (exact contiguous tensors,
// None, addresses, ints that fit; a stream as None, a handle or a stream object) is left to the general path: the functions
// then return NotImplemented and have done nothing.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <limits>
#include <tuple>
#include <type_traits>

#include "../../include/ep.h"

namespace {

PyTypeObject *address_type = nullptr;  // binding.Address

const at::Tensor *plain_tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  return t.layout() == c10::kStrided && t.is_contiguous() ? &t : nullptr;
}

struct Args {
  PyObject *const *a;
  bool plain = true;

  void *pointer(size_t i) {
    PyObject *o = a[i];
    if (o == Py_None) return nullptr;
    if (const at::Tensor *t = plain_tensor(o)) return t->data_ptr();
    if (address_type && Py_TYPE(o) == address_type) return word(o);
    plain = false;
    return nullptr;
  }
  void *handle(size_t i) { return PyLong_CheckExact(a[i]) ? word(a[i]) : refuse(); }
  void *stream(size_t i) {
    if (a[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
    if (PyLong_CheckExact(a[i])) return word(a[i]);
    PyObject *s = PyObject_GetAttrString(a[i], "cuda_stream");
    if (!s) PyErr_Clear();
    void *p = s && PyLong_CheckExact(s) ? word(s) : refuse();
    Py_XDECREF(s);
    return p;
  }
  long long number(size_t i, long long lowest, long long highest) {
    int overflow = 0;
    const long long v = PyLong_CheckExact(a[i]) ? PyLong_AsLongLongAndOverflow(a[i], &overflow) : (plain = false, 0);
    if (overflow || v < lowest || v > highest) plain = false;
    return v;
  }

 private:
  void *refuse() {
    plain = false;
    return nullptr;
  }
  void *word(PyObject *o) {
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) {
      PyErr_Clear();
      plain = false;
    }
    return p;
  }
};

// Parameter i of n: the handle comes first, the stream last.
template <class T>
T convert(Args &in, size_t i, size_t n) {
  if constexpr (std::is_same_v<T, ep_handle *>) return (ep_handle *)in.handle(i);
  else if constexpr (std::is_pointer_v<T>) return (T)(i + 1 == n ? in.stream(i) : in.pointer(i));
  else return (T)in.number(i, std::numeric_limits<T>::min(), std::numeric_limits<T>::max());
}

template <class... A, size_t... I>
PyObject *run(int (*f)(A...), PyObject *const *a, std::index_sequence<I...>) {
  Args in{a};
  int rc = 0;
  std::exception_ptr thrown;
  try {
    const std::tuple<A...> v{convert<A>(in, I, sizeof...(A))...};
    if (!in.plain) Py_RETURN_NOTIMPLEMENTED;
    Py_BEGIN_ALLOW_THREADS
    try {  // (what the library throws must not pass the line that takes the interpreter's lock back)
      rc = std::apply(f, v);
    } catch (...) {
      thrown = std::current_exception();
    }
    Py_END_ALLOW_THREADS
  } catch (...) {  // (from torch: the general path meets the same and reports it)
    Py_RETURN_NOTIMPLEMENTED;
  }
  if (!thrown) return PyLong_FromLong(rc);
  try {
    std::rethrow_exception(thrown);
  } catch (const std::exception &e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    PyErr_SetString(PyExc_RuntimeError, "exception out of the library");
  }
  return nullptr;
}
template <class... A>
PyObject *run(int (*f)(A...), PyObject *const *a, Py_ssize_t n) {
  if (n != (Py_ssize_t)sizeof...(A)) Py_RETURN_NOTIMPLEMENTED;
  return run(f, a, std::index_sequence_for<A...>{});
}
template <auto F>
PyObject *call(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(F, a, n);
}

// row(t, i): what stands for the address of t[i] - t itself for row 0, else an Address.
PyObject *row(PyObject *, PyObject *const *a, Py_ssize_t n) {
  try {
    const at::Tensor *t = n == 2 && address_type && PyLong_CheckExact(a[1]) ? plain_tensor(a[0]) : nullptr;
    int overflow = 0;
    const long long i = t ? PyLong_AsLongLongAndOverflow(a[1], &overflow) : -1;
    if (!t || overflow || t->dim() < 1 || i < 0 || i >= t->size(0)) Py_RETURN_NOTIMPLEMENTED;
    if (i == 0) {
      Py_INCREF(a[0]);
      return a[0];
    }
    char *p = (char *)t->data_ptr() + i * t->stride(0) * (long long)t->element_size();
    PyObject *v = PyLong_FromVoidPtr(p);
    PyObject *r = v ? PyObject_CallOneArg((PyObject *)address_type, v) : nullptr;
    Py_XDECREF(v);
    return r;
  } catch (...) {
    Py_RETURN_NOTIMPLEMENTED;
  }
}

PyObject *set_address_type(PyObject *, PyObject *type) {
  if (!PyType_Check(type) || !PyType_IsSubtype((PyTypeObject *)type, &PyLong_Type)) {
    PyErr_SetString(PyExc_TypeError, "a subclass of int is needed");
    return nullptr;
  }
  Py_INCREF(type);
  Py_XDECREF((PyObject *)address_type);
  address_type = (PyTypeObject *)type;
  Py_RETURN_NONE;
}

#define EP_CALL(f) {#f, (PyCFunction)(void (*)(void))call<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {EP_CALL(ep_layout),
                         EP_CALL(ep_dispatch),
                         EP_CALL(ep_combine),
                         EP_CALL(ep_recv_wait),
                         EP_CALL(ep_fp8_unpack),
                         EP_CALL(ep_ht_dispatch),
                         EP_CALL(ep_dedup),
                         EP_CALL(ep_gather_index),
                         EP_CALL(ep_combine_partial),
                         {"row", (PyCFunction)(void (*)(void))row, METH_FASTCALL, nullptr},
                         {"set_address_type", set_address_type, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
// The torch that this was built for (the binding asks: another one's tensors may be laid out otherwise).
constexpr char built_for[] = "torch " EP_TORCH;
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_epcall", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__epcall(void) {
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", built_for)) Py_CLEAR(m);
  return m;
}
