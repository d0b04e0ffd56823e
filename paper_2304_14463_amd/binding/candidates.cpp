// What the Python binding does before and behind a call of the C ABI, natively: the candidate tensors checked and
// turned into pointers, the result tensor made.  Small calls are bound by the host: a population of 1024 on a graph of
// 50 nodes takes the GPU 4 us, and 8.1 us a call with this part in Python, 6.0 with it here.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <stdint.h>

#include "moccasin.h"

namespace {

using CandidateCall = int (*)(const void* g, int64_t B, const void* starts, const void* ends, const void* active, void* out, void* stream);

[[noreturn]] void refuse(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw python_error();
}

const at::Tensor& tensor(PyObject* x) {
  if (!THPVariable_Check(x)) refuse(PyExc_TypeError, "candidate arrays must be torch tensors");
  return THPVariable_Unpack(x);
}

bool holds(const at::Tensor& x, at::ScalarType type, int64_t n) {
  return x.is_cuda() && x.scalar_type() == type && x.is_contiguous() && x.numel() == n;
}

// A Python int, or None: 0.
uintptr_t address(PyObject* x) {
  if (x == Py_None) return 0;
  const unsigned long long v = PyLong_AsUnsignedLongLong(x);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) throw python_error();
  return (uintptr_t)v;
}

struct Candidates {
  int64_t B;
  const void *starts, *ends, *active;
};
Candidates candidates(int64_t T, const at::Tensor& s, const at::Tensor& e, const at::Tensor& a) {
  const int64_t B = T ? s.numel() / T : 0, n = B * T;
  if (!holds(s, at::kInt, n) || !holds(e, at::kInt, n) || !holds(a, at::kByte, n))
    refuse(PyExc_ValueError, "candidate arrays must be contiguous CUDA tensors [B][T]: int32, int32, uint8");
  return Candidates{B, s.data_ptr(), e.data_ptr(), a.data_ptr()};
}

// pointers(T, starts, ends, active) -> (B, starts, ends, active as addresses); ends None: not looked at, address 0.
PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  if (count != 4) refuse(PyExc_TypeError, "pointers: four arguments");
  const int64_t T = (int64_t)address(args[0]);
  const bool with_ends = args[2] != Py_None;
  const at::Tensor &starts = tensor(args[1]), &active = tensor(args[3]);
  Candidates c = candidates(T, starts, with_ends ? tensor(args[2]) : starts, active);
  if (!with_ends) c.ends = nullptr;
  return Py_BuildValue("LKKK", (long long)c.B, (unsigned long long)(uintptr_t)c.starts, (unsigned long long)(uintptr_t)c.ends,
                       (unsigned long long)(uintptr_t)c.active);
  END_HANDLE_TH_ERRORS
}

// empty(like, bytes of an element: 1 or 4, dimensions..) -> (a new tensor of bytes or of int32 on the device of `like`, its address)
PyObject* empty(PyObject*, PyObject* const* args, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  if (count < 3 || count > 5) refuse(PyExc_TypeError, "empty: three to five arguments");
  int64_t dims[3];
  for (Py_ssize_t i = 2; i < count; ++i) {
    dims[i - 2] = PyLong_AsLongLong(args[i]);
    if (dims[i - 2] == -1 && PyErr_Occurred()) throw python_error();
  }
  const auto options = tensor(args[0]).options().dtype(address(args[1]) == 4 ? at::kInt : at::kByte);
  const at::Tensor made = at::empty(at::IntArrayRef(dims, (size_t)(count - 2)), options);
  THPObjectPtr held(THPVariable_Wrap(made));
  if (!held) throw python_error();
  return Py_BuildValue("NK", held.release(), (unsigned long long)(uintptr_t)made.data_ptr());
  END_HANDLE_TH_ERRORS
}

// evaluate(function, handle, T, starts, ends, active, out or None, per, bytes, stream) -> (code, out): the calls that
// take a batch and leave `per` records of `bytes` bytes per candidate (0: one record, without a dimension of its own).
PyObject* evaluate(PyObject*, PyObject* const* args, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  if (count != 10) refuse(PyExc_TypeError, "evaluate: ten arguments");
  const auto call = reinterpret_cast<CandidateCall>(address(args[0]));
  const void* const handle = reinterpret_cast<const void*>(address(args[1]));
  const at::Tensor& starts = tensor(args[3]);
  const Candidates c = candidates((int64_t)address(args[2]), starts, tensor(args[4]), tensor(args[5]));
  const int64_t per = (int64_t)address(args[7]), bytes = (int64_t)address(args[8]);
  void* const stream = reinterpret_cast<void*>(address(args[9]));
  PyObject* result = args[6];
  if (result == Py_None) {
    const auto options = starts.options().dtype(at::kByte);
    result = THPVariable_Wrap(per ? at::empty({c.B, per, bytes}, options) : at::empty({c.B, bytes}, options));
  } else {
    Py_INCREF(result);
  }
  THPObjectPtr held(result);
  if (!held) throw python_error();
  void* out;
  if (THPVariable_Check(result)) {
    out = THPVariable_Unpack(result).data_ptr();
  } else {   // anything that says where it lies, a storage for one
    THPObjectPtr at(PyObject_CallMethod(result, "data_ptr", nullptr));
    if (!at) throw python_error();
    out = reinterpret_cast<void*>(address(at));
  }
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = call(handle, c.B, c.starts, c.ends, c.active, out, stream);
  Py_END_ALLOW_THREADS
  return Py_BuildValue("iN", code, held.release());
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(pointers)), METH_FASTCALL, nullptr},
                         {"evaluate", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(evaluate)), METH_FASTCALL, nullptr},
                         {"empty", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(empty)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_candidates", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// abi_version: of the header that this was built with.
PyMODINIT_FUNC PyInit__candidates() {
  PyObject* const made = PyModule_Create(&module);
  if (made && PyModule_AddIntConstant(made, "abi_version", MOC_ABI_VERSION) != 0) {
    Py_DECREF(made);
    return nullptr;
  }
  return made;
}
