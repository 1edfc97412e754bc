// The MTTKRP call on torch tensors, natively: argument checks, the current stream and the call into libhbcsf.so in one step.
// The same in Python takes 5 us or so, as long as the kernels of a small tensor's mode: all three modes of 10 000 nonzeros
// 37.6 -> 24.0 us, of 80 000 38.4 -> 26.5 us, most of what is left being the launches.  Only calls that are right are
// carried out here: for any other (and for arguments of any other kind) the caller goes through its own checks, which
// say what is wrong.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "hbcsf.h"

namespace {

// The tensor of a strong type, or null.
const at::Tensor* tensor_of(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool is_matrix(const at::Tensor& t, int64_t rows, int64_t rank, at::ScalarType type) {
  return t.is_cuda() && t.layout() == at::kStrided && t.scalar_type() == type && t.dim() == 2 && t.size(0) == rows &&
         t.size(1) == rank && t.is_contiguous();
}

// mttkrp(handle, dims, mode, factors, out) -> out, or an error code of the library, or None: not a call for this path.
PyObject* mttkrp(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 5 || !PyLong_CheckExact(args[0]) || !PyTuple_CheckExact(args[1]) || !PyLong_CheckExact(args[2]) ||
      !(PyList_CheckExact(args[3]) || PyTuple_CheckExact(args[3])))
    Py_RETURN_NONE;
  const Py_ssize_t order = PyTuple_GET_SIZE(args[1]);
  const long mode = PyLong_AsLong(args[2]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (order > HBCSF_MAX_ORDER || mode < 0 || mode >= order || PySequence_Fast_GET_SIZE(args[3]) < order) Py_RETURN_NONE;
  int64_t dims[HBCSF_MAX_ORDER];
  for (Py_ssize_t m = 0; m < order; ++m) dims[m] = PyLong_AsLongLong(PyTuple_GET_ITEM(args[1], m));
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  PyObject** items = PySequence_Fast_ITEMS(args[3]);
  const void* ptrs[HBCSF_MAX_ORDER] = {};
  const at::Tensor* first = nullptr;
  for (Py_ssize_t m = 0; m < order; ++m) {
    if (m == mode) continue;
    const at::Tensor* f = tensor_of(items[m]);
    if (!f || f->dim() != 2) Py_RETURN_NONE;
    if (!first) first = f;
    if (!is_matrix(*f, dims[m], first->size(1), first->scalar_type())) Py_RETURN_NONE;
    ptrs[m] = f->data_ptr();
  }
  if (!first) Py_RETURN_NONE;
  const at::ScalarType type = first->scalar_type();
  const int64_t rank = first->size(1);
  if ((type != at::kFloat && type != at::kDouble) || rank > 1024) Py_RETURN_NONE;
  at::Tensor made;
  const at::Tensor* out = &made;
  if (args[4] == Py_None) {
    made = at::empty({dims[mode], rank}, at::TensorOptions(type).device(at::Device(at::kCUDA, c10::hip::current_device())));
  } else {
    out = tensor_of(args[4]);
    if (!out || !is_matrix(*out, dims[mode], rank, type)) Py_RETURN_NONE;
  }
  void* handle = PyLong_AsVoidPtr(args[0]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  void* to = out->data_ptr();
  void* stream = c10::hip::getCurrentHIPStream().stream();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = type == at::kFloat
           ? hbcsf_mttkrp((const hbcsf_tensor*)handle, (int)mode, (int)rank, (const float* const*)ptrs, (float*)to, stream)
           : hbcsf_mttkrp_f64((const hbcsf_tensor*)handle, (int)mode, (int)rank, (const double* const*)ptrs, (double*)to, stream);
  Py_END_ALLOW_THREADS
  if (rc != HBCSF_OK) return PyLong_FromLong(rc);
  if (args[4] == Py_None) return THPVariable_Wrap(std::move(made));
  Py_INCREF(args[4]);
  return args[4];
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"mttkrp", (PyCFunction)(void (*)(void))mttkrp, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hbcsf_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The tensors' layout is that of the torch this was compiled against: under any other the module does not load.
PyMODINIT_FUNC PyInit__hbcsf_torch() {
  PyObject* torch = PyImport_ImportModule("torch");
  PyObject* version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
  const char* text = version ? PyUnicode_AsUTF8(version) : nullptr;
  const bool same = text && std::strcmp(text, HBCSF_TORCH) == 0;
  if (text && !same) PyErr_Format(PyExc_ImportError, "built for torch " HBCSF_TORCH ", this is torch %s", text);
  Py_XDECREF(version);
  Py_XDECREF(torch);
  return same ? PyModule_Create(&module) : nullptr;
}
