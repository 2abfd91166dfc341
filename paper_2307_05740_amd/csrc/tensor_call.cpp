// The repeated calls of the Python classes on torch tensors without the interpreter's detour: a call asks each
// tensor what it is and starts the product in native code.  A product over a few thousand rows takes the GPU 3.4 to
// 4.5 us; asked one attribute at a time and called through ctypes it took the host 4.7 to 5.2 us, of which the launch
// itself is 2.4.
//
// Every function returns 1 where it has called the library and that has accepted, the library's error code (negative)
// where it has not, and 0 where the arguments are anything but the plain case: dense float32 tensors of the
// right sizes on the handle's device.  The caller then goes the general way, which allocates, asserts and reports.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

// The tensor where it is a dense, contiguous float32 one on the device, else null.
const at::Tensor* plain(PyObject* o, int64_t device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.has_storage() || t.scalar_type() != at::kFloat || !t.is_cuda() || t.get_device() != device || !t.is_contiguous())
    return nullptr;
  return &t;
}

const at::Tensor* matrix(PyObject* o, int64_t device, int64_t rows) {
  const at::Tensor* t = plain(o, device);
  return t && t->dim() == 2 && t->size(0) == rows ? t : nullptr;
}

bool integers(PyObject* const* args, int count, int64_t* out) {
  for (int i = 0; i < count; ++i) {
    out[i] = PyLong_AsLongLong(args[i]);
    if (out[i] == -1 && PyErr_Occurred()) return false;
  }
  return true;
}

float* at_data(const at::Tensor* t) { return static_cast<float*>(t->data_ptr()); }
void* stream_of(int64_t device) { return c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream(); }

template <typename F>
PyObject* guarded(F&& call) {
  try {
    return PyLong_FromLong(call());
  } catch (...) {             // (a tensor without data: the general way says what is wrong with it)
    return PyLong_FromLong(0);
  }
}

template <typename F>
long started(F&& call) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return rc == 0 ? 1 : rc;
}

bool arguments(Py_ssize_t have, Py_ssize_t want) {
  if (have != want) PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, have);
  return have == want;
}

// spmm(function, handle, device, n, most columns, X, Y)
PyObject* spmm(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  int64_t v[5];
  if (!arguments(n_args, 7) || !integers(args, 5, v)) return nullptr;
  return guarded([&]() -> long {
    const at::Tensor *X = matrix(args[5], v[2], v[3]), *Y = matrix(args[6], v[2], v[3]);
    if (!X || !Y || X->size(1) != Y->size(1) || X->size(1) < 1 || X->size(1) > v[4]) return 0;
    auto call = reinterpret_cast<int (*)(void*, const float*, float*, int32_t, void*)>(v[0]);
    float *x = at_data(X), *y = at_data(Y);
    const int32_t k = (int32_t)X->size(1);
    void* stream = stream_of(v[2]);
    return started([&] { return call(reinterpret_cast<void*>(v[1]), x, y, k, stream); });
  });
}

// sddmm(function, handle, device, n, most columns, entries, U, V, S)
PyObject* sddmm(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  int64_t v[6];
  if (!arguments(n_args, 9) || !integers(args, 6, v)) return nullptr;
  return guarded([&]() -> long {
    const at::Tensor *U = matrix(args[6], v[2], v[3]), *V = matrix(args[7], v[2], v[3]), *S = plain(args[8], v[2]);
    if (!U || !V || !S || U->size(1) != V->size(1) || U->size(1) < 1 || U->size(1) > v[4] || S->numel() != v[5]) return 0;
    auto call = reinterpret_cast<int (*)(void*, const float*, const float*, float*, int32_t, void*)>(v[0]);
    float *u = at_data(U), *w = at_data(V), *s = at_data(S);
    const int32_t k = (int32_t)U->size(1);
    void* stream = stream_of(v[2]);
    return started([&] { return call(reinterpret_cast<void*>(v[1]), u, w, s, k, stream); });
  });
}

// mttkrp(function, handle, device, I, J, K, most columns, B, C, A)
PyObject* mttkrp(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  int64_t v[7];
  if (!arguments(n_args, 10) || !integers(args, 7, v)) return nullptr;
  return guarded([&]() -> long {
    const at::Tensor *B = matrix(args[7], v[2], v[4]), *C = matrix(args[8], v[2], v[5]), *A = matrix(args[9], v[2], v[3]);
    if (!A || !B || !C || B->size(1) != A->size(1) || C->size(1) != A->size(1) || A->size(1) < 1 || A->size(1) > v[6]) return 0;
    auto call = reinterpret_cast<int (*)(void*, const float*, const float*, float*, int32_t, void*)>(v[0]);
    float *a = at_data(A), *b = at_data(B), *c = at_data(C);
    const int32_t R = (int32_t)A->size(1);
    void* stream = stream_of(v[2]);
    return started([&] { return call(reinterpret_cast<void*>(v[1]), b, c, a, R, stream); });
  });
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<spmm>("spmm"), method<sddmm>("sddmm"), method<mttkrp>("mttkrp"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "tensor_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_tensor_call() { return PyModule_Create(&module); }
