// The calls of the Linear from Python in one native function: what `ams_linear` and its variants in __init__.py check of their
// tensors, the current stream and the call of libams.so, with the interpreter left out.  An eager call of 256 x 768 is bound
// by this (the kernel takes 2.3 us).  It takes plain tensors and integers and answers None to everything else, and to a call that the library
// refuses: the caller then goes the long way, which raises what there is to raise.
//
// It is not linked to libams.so but given the addresses of the entry points of the one that the package has loaded: a path or a
// name in the dynamic section could find another tree's.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include <cxxabi.h>
#include <string.h>

#include "../../include/ams.h"

namespace {

// A plain strided tensor on the current GPU (the kernels run there, in the order of its stream): no subclass, no wrapper of a
// transformation, no view that needs resolving.
const at::Tensor* plain(PyObject* o, c10::ScalarType type, c10::DeviceIndex device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined()) return nullptr;
  constexpr auto ordinary =
      c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
  if ((t.key_set().raw_repr() & ~ordinary.raw_repr()) != 0 || !t.is_cuda() || t.get_device() != device || t.scalar_type() != type || !t.is_contiguous()) return nullptr;
  return &t;
}

bool whole(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &overflow);
  return !overflow;
}

enum Entry { kPlain, kWorkspace, kStatic, kGrouped };

// The entry points that are called, in the order in which bind() takes them.
struct Library {
  decltype(&ams_packed_bytes) packed_bytes;
  decltype(&ams_group_scales_count) group_scales_count;
  decltype(&ams_linear) linear;
  decltype(&ams_linear_ws) linear_ws;
  decltype(&ams_linear_static_ws) linear_static_ws;
  decltype(&ams_linear_grouped) linear_grouped;
} lib;

// bind(address of each entry point of Library)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* at[6];
  if (n != 6) return PyErr_Format(PyExc_TypeError, "bind takes 6 addresses");
  for (int i = 0; i < 6; i++)
    if (!(at[i] = PyLong_AsVoidPtr(a[i]))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "no address");
  static_assert(sizeof lib == sizeof at, "one address for each");
  memcpy(&lib, at, sizeof lib);
  Py_RETURN_NONE;
}

// What a call of the library takes.
struct Call {
  int64_t entry, M, N, K, group;
  int fmt;
  const void* w;
  const uint16_t *s, *x;
  uint16_t* y;
  void* ws;
  size_t ws_bytes;
  void* st;
};

// linear's arguments, checked; false for those that are not taken.
bool arguments(PyObject* const* a, Py_ssize_t n, Call* c) try {
  int64_t entry = 0, N = 0, fmt = 0, group = 0;
  if (!lib.linear || n != 8 || !whole(a[0], &entry) || !whole(a[4], &N) || !whole(a[5], &fmt)) return false;
  if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) return false;
  const auto stream = c10::hip::getCurrentHIPStream();  // of the current device
  const c10::DeviceIndex dev = stream.device_index();
  const at::Tensor *W = plain(a[1], at::kByte, dev), *scales = plain(a[2], at::kHalf, dev), *X = plain(a[3], at::kHalf, dev), *out = plain(a[6], at::kHalf, dev);
  if (!W || !scales || !X || !out || X->dim() != 2 || fmt < 0 || fmt > 0x7FFF) return false;
  const int64_t M = X->size(0), K = X->size(1);
  if (M > AMS_MAX_M || N <= 0 || N > (1 << 24) || out->numel() < M * N) return false;
  size_t bytes = 0, count = 0;
  if (lib.packed_bytes((int)fmt, N, K, &bytes) != AMS_OK || (size_t)W->numel() != bytes) return false;
  const at::Tensor* workspace = nullptr;
  if (entry == kGrouped) {
    if (!whole(a[7], &group) || lib.group_scales_count((int)fmt, N, K, group, &count) != AMS_OK || (size_t)scales->numel() != count) return false;
  } else {
    if (scales->numel() != N) return false;
    if (entry == kWorkspace && a[7] != Py_None && !(workspace = plain(a[7], at::kByte, dev))) return false;
  }
  *c = {entry, M, N, K, group, (int)fmt, W->const_data_ptr(), (const uint16_t*)scales->const_data_ptr(), (const uint16_t*)X->const_data_ptr(), (uint16_t*)out->data_ptr(),
        workspace ? workspace->data_ptr() : nullptr, workspace ? (size_t)workspace->numel() : 0, (void*)stream.stream()};
  return true;
} catch (...) {  // torch's own checks; the long way meets them again
  return false;
}

int call(const Call& c) {
  switch (c.entry) {
    case kPlain: return lib.linear(c.w, c.s, c.x, c.y, (int)c.M, c.N, c.K, c.fmt, c.st);
    case kWorkspace: return lib.linear_ws(c.w, c.s, c.x, c.y, (int)c.M, c.N, c.K, c.fmt, c.ws, c.ws_bytes, c.st);
    case kStatic: return lib.linear_static_ws(c.w, c.s, c.x, c.y, (int)c.M, c.N, c.K, c.fmt, c.st);
    case kGrouped: return lib.linear_grouped(c.w, c.s, c.group, c.x, c.y, (int)c.M, c.N, c.K, c.fmt, c.st);
  }
  return -1;
}

// The call, with the interpreter's lock given up for it.  It is taken again outside of every try block and destructor: where the
// interpreter ends meanwhile, pthread_exit ends a daemon thread there by unwinding its stack, and a handler that stops that, or
// a destructor that it would leave, aborts the process.
int call_unlocked(const Call& c) {
  PyThreadState* const state = PyEval_SaveThread();
  int rc = -1;
  try {
    rc = call(c);
  } catch (const abi::__forced_unwind&) {
    throw;
  } catch (...) {
  }
  PyEval_RestoreThread(state);
  return rc;
}

// linear(entry, W_packed, scales, X, N, fmt, out, workspace or scale_group): out, or None.
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Call c;
  if (!arguments(a, n, &c) || call_unlocked(c) != AMS_OK) Py_RETURN_NONE;
  Py_INCREF(a[6]);
  return a[6];
}

PyMethodDef methods[] = {{"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
                         {"linear", (PyCFunction)(void (*)(void))linear, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  PyObject* const m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "BUILT_FOR", AMS_TORCH) != 0) {  // whose tensors it reads
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
