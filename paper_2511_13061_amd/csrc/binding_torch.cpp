// The product and conversion calls of the Python binding as native functions: what they do between the caller and the C ABI
// (an output tensor, its address, the current stream) takes 2.4 us of a 5.8 us call in Python, and a small product is over
// on the GPU in 3.4.  Only plain device tensors and the current stream are served; for anything else the functions return None and
// the caller goes the general way through ctypes.  They call the entry points of the libmacko.so that is loaded already
// (bind() is given their addresses), and release the interpreter's lock around allocation and call, as ctypes does.
//
// Per call, through ctypes and here: a 512 x 512 product 5.8 and 4.9 us, a small batch product 7.8 and 5.6, a small decode 7.2 and
// 5.1.  Of the 4.9: 3.2 the runtime's launch (of an empty kernel as well), 0.2 the rest of the library, 0.3 the function
// here, 0.9 to 1.0 the output tensor (none if the caller gives one), 0.2 Python.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <pthread.h>

#include <algorithm>
#include <cstdint>

#include "macko.h"

namespace {

decltype(&macko_spmv) g_spmv = nullptr;
decltype(&macko_spmm) g_spmm = nullptr;
decltype(&macko_decode_device) g_decode = nullptr;

// A forked child may not use its parent's device.  PyTorch's Python calls refuse that with an error, the C++ calls below do not:
// in a child the functions serve nothing, and the general way says what there is to say.
bool g_forked = false;

// A plain tensor on the GPU (no subclass: those may define what their methods do).
const at::Tensor* device_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() ? &t : nullptr;
}

// What a call returns: its status as a number if it failed, else the tensor.
PyObject* result(int status, const at::Tensor& made, PyObject* given) {
  if (status != MACKO_OK) return PyLong_FromLong(status);
  if (given != Py_None) return Py_NewRef(given);
  return THPVariable_Wrap(made);
}

bool handle_of(PyObject* o, macko_handle_t* h) {       // None: a handle that has been destroyed
  *h = o == Py_None ? nullptr : static_cast<macko_handle_t>(PyLong_AsVoidPtr(o));
  return !PyErr_Occurred();
}

// spmv(handle, rows, x, y or None)
PyObject* spmv(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4) return PyErr_Format(PyExc_TypeError, "4 arguments");
  const at::Tensor* x = device_tensor(args[2]);
  const at::Tensor* given = args[3] == Py_None ? nullptr : device_tensor(args[3]);
  if (!g_spmv || g_forked || !x || (args[3] != Py_None && !given)) Py_RETURN_NONE;
  macko_handle_t h;
  if (!handle_of(args[0], &h)) return nullptr;
  const int64_t rows = PyLong_AsLongLong(args[1]);
  if (PyErr_Occurred()) return nullptr;
  at::Tensor y;
  int status;
  {
    pybind11::gil_scoped_release unlocked;
    if (!given) y = at::empty({rows}, at::TensorOptions().dtype(at::kHalf).device(x->device()));
    status = g_spmv(h, x->data_ptr(), (given ? *given : y).data_ptr(), c10::hip::getCurrentHIPStream().stream());
  }
  return result(status, y, args[3]);
  END_HANDLE_TH_ERRORS
}

// spmm(handle, rows, X, Y or None)
PyObject* spmm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4) return PyErr_Format(PyExc_TypeError, "4 arguments");
  const at::Tensor* x = device_tensor(args[2]);
  const at::Tensor* given = args[3] == Py_None ? nullptr : device_tensor(args[3]);
  if (!g_spmm || g_forked || !x || (args[3] != Py_None && !given)) Py_RETURN_NONE;
  if (x->dim() != 2 || x->stride(1) != 1 || x->size(0) > MACKO_MAX_BATCH || (given && given->dim() != 2)) Py_RETURN_NONE;
  macko_handle_t h;
  if (!handle_of(args[0], &h)) return nullptr;
  const int64_t rows = PyLong_AsLongLong(args[1]), batch = x->size(0);
  if (PyErr_Occurred()) return nullptr;
  at::Tensor made;
  int status;
  {
    pybind11::gil_scoped_release unlocked;
    if (!given) made = at::empty({batch, rows}, at::TensorOptions().dtype(at::kHalf).device(x->device()));
    const at::Tensor& y = given ? *given : made;
    const int64_t ldx = batch > 1 ? x->stride(0) : std::max<int64_t>(x->size(1), 1);
    const int64_t ldy = batch > 1 ? y.stride(0) : std::max<int64_t>(y.size(1), 1);
    status = g_spmm(h, (int)batch, x->data_ptr(), ldx, y.data_ptr(), ldy, c10::hip::getCurrentHIPStream().stream());
  }
  return result(status, made, args[3]);
  END_HANDLE_TH_ERRORS
}

// decode_device(handle, rows, cols, bits per value): into a new tensor on the current device
PyObject* decode_device(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4) return PyErr_Format(PyExc_TypeError, "4 arguments");
  if (!g_decode || g_forked) Py_RETURN_NONE;
  macko_handle_t h;
  if (!handle_of(args[0], &h)) return nullptr;
  const int64_t rows = PyLong_AsLongLong(args[1]), cols = PyLong_AsLongLong(args[2]), bits = PyLong_AsLongLong(args[3]);
  if (PyErr_Occurred()) return nullptr;
  at::Tensor dense;
  int status;
  {
    pybind11::gil_scoped_release unlocked;
    dense = at::empty({rows, cols}, at::TensorOptions().dtype(bits == 8 ? at::kByte : at::kHalf).device(at::kCUDA));
    status = g_decode(h, dense.data_ptr(), rows > 1 ? dense.stride(0) : std::max<int64_t>(cols, 1), c10::hip::getCurrentHIPStream().stream());
  }
  return result(status, dense, Py_None);
  END_HANDLE_TH_ERRORS
}

// bind(address of macko_spmv, of macko_spmm, of macko_decode_device)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) return PyErr_Format(PyExc_TypeError, "3 arguments");
  void* p[3];
  for (int i = 0; i < 3; ++i) p[i] = PyLong_AsVoidPtr(args[i]);
  if (PyErr_Occurred()) return nullptr;
  if (!g_spmv && pthread_atfork(nullptr, nullptr, [] { g_forked = true; }) != 0) return PyErr_NoMemory();
  g_spmv = reinterpret_cast<decltype(g_spmv)>(p[0]);
  g_spmm = reinterpret_cast<decltype(g_spmm)>(p[1]);
  g_decode = reinterpret_cast<decltype(g_decode)>(p[2]);
  Py_RETURN_NONE;
}

#define MACKO_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MACKO_FAST(spmv), MACKO_FAST(spmm), MACKO_FAST(decode_device), MACKO_FAST(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
