// The per-layer calls of Cache (binding.py) from Python without ctypes: a module of one function, which looks at the tensors and
// calls the C entry point.  A decode step of a small cache takes the GPU less than the checks and conversions of the same call took
// in Python.
//
// call(entry, handle, layer, tensors, q_row, kv_row, device, stream, token_begin) -> the entry point's code, or None where anything
// about the arguments is not plainly as it should be: the caller then takes its Python path, which has the same checks and says what is
// wrong.  Nothing is kept from one call to the next, and no C++ exception leaves: what a tensor throws when it is looked at counts as not plain.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

// where the tensors have to be (the tests build the module for the CPU, too)
#ifndef KVP_TENSOR_DEVICE
#define KVP_TENSOR_DEVICE c10::DeviceType::CUDA
#endif

namespace {

constexpr int kMostTensors = 5;

// a plain contiguous bf16 tensor of `device`; its address is then what data_ptr() gives
bool plain(PyObject* o, int64_t device, const at::Tensor** out) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.is_nested()) return false;
  const auto keys = t.key_set();
  if (keys.has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                        c10::DispatchKey::Functionalize, c10::DispatchKey::Batched, c10::DispatchKey::ZeroTensor})))
    return false;
  if (t.layout() != at::kStrided || !t.has_storage() || t.scalar_type() != at::kBFloat16 || !t.is_contiguous()) return false;
  const c10::Device d = t.device();
  if (d.type() != KVP_TENSOR_DEVICE || d.index() != device) return false;
  *out = &t;
  return true;
}

bool small_int(PyObject* o, int32_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) return false;
  *out = (int32_t)v;
  return true;
}

bool address(PyObject* o, void** out) {
  if (!PyLong_CheckExact(o)) return false;
  const unsigned long long v = PyLong_AsUnsignedLongLong(o);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *out = (void*)(uintptr_t)v;
  return true;
}

bool pair(PyObject* o, int64_t (&out)[2]) {
  if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 2) return false;
  for (int i = 0; i < 2; ++i) {
    int32_t v;
    if (!small_int(PyTuple_GET_ITEM(o, i), &v)) return false;
    out[i] = v;
  }
  return true;
}

bool rows_of(const at::Tensor& t, const int64_t (&row)[2], int64_t rows) {       // [rows, row[0], row[1]]
  return t.dim() == 3 && t.size(0) == rows && t.size(1) == row[0] && t.size(2) == row[1];
}

// the tensors' addresses, the rows of K and those of q_obs, where all are plain and of the shapes that belong together
bool plain_tensors(PyObject* list, Py_ssize_t n_tensors, bool step, const int64_t (&q_row)[2], const int64_t (&kv_row)[2], int64_t device,
                   void* (&p)[kMostTensors], int64_t* rows, int64_t* n_obs) {
  const at::Tensor* t[kMostTensors];
  for (Py_ssize_t i = 0; i < n_tensors; ++i) {
    if (!plain(PyTuple_GET_ITEM(list, i), device, &t[i])) return false;
    p[i] = t[i]->numel() > 0 ? t[i]->mutable_data_ptr() : nullptr;
  }
  *rows = t[1]->dim() == 3 ? t[1]->size(0) : -1;
  *n_obs = n_tensors == 5 && t[4]->dim() == 3 ? t[4]->size(0) : 0;
  if (*rows < 0 || *rows > INT32_MAX || *n_obs > INT32_MAX || !rows_of(*t[1], kv_row, *rows) || !rows_of(*t[2], kv_row, *rows)) return false;
  for (const int i : {0, 3}) {
    if (step ? t[i]->dim() != 2 || t[i]->size(0) != q_row[0] || t[i]->size(1) != q_row[1] : !rows_of(*t[i], q_row, *rows)) return false;
  }
  return n_tensors < 5 || rows_of(*t[4], q_row, *n_obs);
}

// `tensors`: (q, k_tail, v_tail, out) of a step, token_begin None; or (q, k, v, out[, q_obs]) of a block
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  if (n_args != 9) {
    PyErr_SetString(PyExc_TypeError, "call takes nine arguments");
    return nullptr;
  }
  void *entry, *handle, *stream;
  int32_t layer, device, token_begin = 0;
  int64_t q_row[2], kv_row[2];
  PyObject* const list = args[3];
  const bool step = args[8] == Py_None;
  if (!address(args[0], &entry) || !entry || !address(args[1], &handle) || !handle || !small_int(args[2], &layer) || !PyTuple_CheckExact(list) ||
      !pair(args[4], q_row) || !pair(args[5], kv_row) || !small_int(args[6], &device) || !address(args[7], &stream) ||
      (!step && !small_int(args[8], &token_begin)))
    Py_RETURN_NONE;
  const Py_ssize_t n_tensors = PyTuple_GET_SIZE(list);
  if (n_tensors < 4 || n_tensors > (step ? 4 : kMostTensors)) Py_RETURN_NONE;
  void* p[kMostTensors];
  int64_t rows = -1, n_obs = 0;
  try {
    if (!plain_tensors(list, n_tensors, step, q_row, kv_row, device, p, &rows, &n_obs)) Py_RETURN_NONE;
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  int code;
  Py_BEGIN_ALLOW_THREADS;                    // (as ctypes does: a launch may have to wait)
  if (step)
    code = ((int (*)(void*, int32_t, const void*, const void*, const void*, int32_t, void*, void*))entry)(handle, layer, p[0], p[1], p[2],
                                                                                                     (int32_t)rows, p[3], stream);
  else if (n_tensors == 4)
    code = ((int (*)(void*, int32_t, int32_t, int32_t, const void*, const void*, const void*, void*, void*))entry)(
        handle, layer, token_begin, (int32_t)rows, p[0], p[1], p[2], p[3], stream);
  else
    code = ((int (*)(void*, int32_t, int32_t, int32_t, const void*, const void*, const void*, void*, const void*, int32_t, void*))entry)(
        handle, layer, token_begin, (int32_t)rows, p[0], p[1], p[2], p[3], p[4], (int32_t)n_obs, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(code);
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: that of the headers the module was built with, whose layouts of a tensor are part of its code
PyMODINIT_FUNC PyInit__fast_calls() {
  PyObject* const m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", KVP_TORCH_VERSION) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
