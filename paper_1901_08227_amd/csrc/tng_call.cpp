// The hot calls of binding.py without a trip through ctypes: an argument check and the call of a C entry point, in one
// extension function.  What bounds a small call is the host: of the 11.5 us that encode + decode of 4 x 25000 gradients took
// back to back, 8.5 were kernels; a pass through the checks in Python and ctypes is 0.5 to 0.7 us a tensor.
//
//   call(address, handle, iter, kinds, d, M, words, tensor, ...) -> status, or None
//
// address: of the entry point; kinds: a letter per tensor, d float32[d], g float32[M d], c int32[M words], s float32[M], behind a
// '-' for an entry point that takes no iteration number (iter is then not looked at).  None says that an argument is not a plain
// case (no tensor, another type, too short, a tensor subclass other than Parameter or a wrapper without storage, an iteration that
// is no int): nothing was called, and the caller goes the way through ctypes, which raises what there is to raise.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

constexpr int kFixed = 7, kMaxTensors = 6;

// True if obj is a plain device tensor of that type and at least n elements; *p is its address (null for None).
bool device_address(PyObject* obj, char kind, int64_t d, int64_t M, int64_t words, void** p) {
  if (obj == Py_None) {
    *p = nullptr;
    return true;
  }
  if (!THPVariable_CheckExact(obj)) return false;
  const at::Tensor& t = THPVariable_Unpack(obj);
  if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous()) return false;
  if (t.scalar_type() != (kind == 'c' ? at::kInt : at::kFloat)) return false;
  const int64_t n = kind == 'd' ? d : kind == 'g' ? M * d : kind == 'c' ? M * words : M;
  if (t.numel() < n) return false;
  *p = t.data_ptr();
  return true;
}

template <typename... P>
int enter(uintptr_t f, void* h, bool with_iter, uint32_t iter, P... p) {
  if (with_iter) return reinterpret_cast<int (*)(void*, uint32_t, P...)>(f)(h, iter, p...);
  return reinterpret_cast<int (*)(void*, P...)>(f)(h, p...);
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  const Py_ssize_t n = nargs - kFixed;
  const char* kinds = nullptr;
  if (n < 2 || n > kMaxTensors || !PyUnicode_Check(args[3]) || (kinds = PyUnicode_AsUTF8(args[3])) == nullptr ||
      PyUnicode_GET_LENGTH(args[3]) != n + (kinds[0] == '-')) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "call: a letter per tensor, 2 to 6 tensors");
    return nullptr;
  }
  const bool with_iter = kinds[0] != '-';
  if (!with_iter) ++kinds;
  // (anything but a plain int as handle or iteration, None too, goes through ctypes, which converts or refuses it)
  if (!PyLong_CheckExact(args[1]) || (with_iter && !PyLong_CheckExact(args[2]))) Py_RETURN_NONE;
  const uintptr_t f = (uintptr_t)PyLong_AsUnsignedLongLong(args[0]);
  void* h = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLong(args[1]));
  const uint32_t iter = with_iter ? (uint32_t)PyLong_AsUnsignedLongMask(args[2]) : 0u;  // (as ctypes does)
  const int64_t d = PyLong_AsLongLong(args[4]), M = PyLong_AsLongLong(args[5]), words = PyLong_AsLongLong(args[6]);
  if (PyErr_Occurred()) return nullptr;
  void* p[kMaxTensors] = {};
  try {
    for (Py_ssize_t i = 0; i < n; ++i)
      if (!device_address(args[kFixed + i], kinds[i], d, M, words, &p[i])) Py_RETURN_NONE;
  } catch (const std::exception&) {  // (an address that cannot be had: ctypes' way says why)
    Py_RETURN_NONE;
  }
  int status = -1;
  Py_BEGIN_ALLOW_THREADS
  switch (n) {
    case 2: status = enter(f, h, with_iter, iter, p[0], p[1]); break;
    case 3: status = enter(f, h, with_iter, iter, p[0], p[1], p[2]); break;
    case 4: status = enter(f, h, with_iter, iter, p[0], p[1], p[2], p[3]); break;
    case 5: status = enter(f, h, with_iter, iter, p[0], p[1], p[2], p[3], p[4]); break;
    default: status = enter(f, h, with_iter, iter, p[0], p[1], p[2], p[3], p[4], p[5]); break;
  }
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyMethodDef methods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "tng_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and Python that this was compiled for (the binding uses it with no other).
PyMODINIT_FUNC PyInit_tng_call() {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", TNG_BUILT_FOR) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
