// Native marshalling of the calls that a program makes per layer.  A small layer's call costs the host more than the device
// (one image through a 384 x 384 projection: 3.8 us of kernel, 7.3 us per call in Python), so a call whose arguments are all
// in the ordinary form -- plain device tensors of the right types and shapes, Python integers -- is read, checked and
// handed to the C ABI here.  Anything else is declined (NotImplemented), and the Python function goes on with it: it
// knows the other forms that are accepted and names what is wrong with the ones that are not.  Nothing is kept
// between calls.
// Measured per call: the projection above 7.3 -> 4.1 us; 768 -> 1000 at 4:8 on 8 tokens, plain, 8.2 -> 6.2 (5.0 with a kernel
// that has become faster since); the twelve calls and sixteen allocations that compress a block by scores and expand it 94 -> 63.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <exception>
#include <optional>

#include "nm_sparse.h"

namespace {

// The C ABI of the library that Python has loaded (set once by bind), and the Python helpers of the rare ways on.
struct Library {
  decltype(&nm_prune) prune;
  decltype(&nm_prune_scored) prune_scored;
  decltype(&nm_pack) pack;
  decltype(&nm_unpack) unpack;
  decltype(&nm_linear_forward) forward;
  decltype(&nm_linear_forward_prepared) forward_prepared;
  decltype(&nm_linear_forward_static) forward_static;
  decltype(&nm_spmm_workspace_bytes) workspace_bytes;
  decltype(&nm_values_bytes) values_bytes;
  decltype(&nm_index_bytes) index_bytes;
  // may be missing: a prepared layer is then multiplied uncut
  decltype(&nm_linear_forward_prepared_scratch) forward_prepared_scratch;
  decltype(&nm_prepared_scratch_bytes) prepared_scratch_bytes;
} lib;
PyObject* raise_status;    // raises NmError for a status that is not NM_OK
PyObject* find_workspace;  // the scratch tensor of a device and stream

PyObject* declined() { Py_RETURN_NOTIMPLEMENTED; }

// A device tensor that is nothing but that: no subclass, no functional transform's wrapper, no lazy conjugate or negation.
bool plain(PyObject* obj, at::ScalarType type, const at::Tensor** out) {
  if (!THPVariable_CheckExact(obj)) return false;
  const at::Tensor& t = THPVariable_Unpack(obj);
  constexpr c10::DispatchKeySet ordinary({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                          c10::DispatchKey::AutocastCUDA});
  if (!t.defined() || t.key_set() - ordinary != c10::DispatchKeySet(c10::BackendComponent::CUDABit) || t.scalar_type() != type ||
      !t.has_storage())
    return false;
  *out = &t;
  return true;
}

bool integer(PyObject* obj, int64_t lo, int64_t hi, int64_t* out) {
  if (!PyLong_CheckExact(obj)) return false;
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(obj, &overflow);
  if (overflow || v < lo || v > hi) return false;
  *out = v;
  return true;
}
bool level(PyObject* n, PyObject* m, int32_t* N, int32_t* M) {
  int64_t a, b;
  if (!integer(n, 0, 16, &a) || !integer(m, 0, 16, &b)) return false;
  *N = (int32_t)a;
  *M = (int32_t)b;
  return true;
}

// rows, columns and leading dimension of a matrix whose rows are contiguous
struct Matrix { int64_t rows, cols, ld; };
bool matrix(const at::Tensor& t, Matrix* m) {
  if (t.dim() != 2) return false;
  m->rows = t.size(0);
  m->cols = t.size(1);
  if (t.stride(1) != 1 && m->cols > 1) return false;
  m->ld = m->rows > 1 ? t.stride(0) : m->cols;
  return true;
}
bool whole(const at::Tensor& t) { return t.dim() == 2 && t.is_contiguous(); }

// The stream of a call: the given one, or the current one of the current device.
bool stream_of(PyObject* obj, void** out) {
  if (obj == Py_None) {
    *out = c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream();
    return true;
  }
  PyObject* handle = PyObject_GetAttrString(obj, "cuda_stream");
  if (handle == nullptr) { PyErr_Clear(); return false; }
  const bool ok = PyLong_CheckExact(handle);
  if (ok) *out = PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  if (PyErr_Occurred()) { PyErr_Clear(); return false; }
  return ok;
}

// Tracing modes and the like see every tensor operation: they get the Python functions.
bool observed() { return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set(); }

template <class T>
T* pointer(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

// f without the interpreter lock: other threads run meanwhile, and a stream's host function that needs it can end.  f allocates
// the outputs, which may free cached memory and wait for the device, and calls the library; the arguments' pointers are taken
// before.  (One release for both: each takes 0.1 us.)  An exception of f goes on when the lock is held again.  Not noexcept: where
// the interpreter has ended meanwhile, taking its lock again ends this thread by unwinding its stack.
template <class F>
auto unlocked(F&& f) {
  std::optional<decltype(f())> r;
  std::exception_ptr failed;
  PyThreadState* self = PyEval_SaveThread();
  try {
    r.emplace(f());
  } catch (...) {
    failed = std::current_exception();
  }
  PyEval_RestoreThread(self);
  if (failed) std::rethrow_exception(failed);
  return *std::move(r);
}
PyObject* result(int32_t st, PyObject* value) {  // steals value
  if (st == NM_OK) return value;
  Py_XDECREF(value);
  PyObject* r = PyObject_CallFunction(raise_status, "i", (int)st);
  Py_XDECREF(r);
  return nullptr;
}

at::Tensor fresh(at::Device device, int64_t rows, int64_t cols, at::ScalarType type) {
  return at::empty({rows, cols}, at::TensorOptions().dtype(type).device(device));
}

// prune(W, N, M, W_masked, stream)
PyObject* prune(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *W, *Wm = nullptr;
  Matrix w, wm;
  int32_t N, M;
  void* s;
  if (n != 5 || observed() || !plain(a[0], at::kBFloat16, &W) || !matrix(*W, &w) || !level(a[1], a[2], &N, &M)) return declined();
  if (a[3] != Py_None &&
      (!plain(a[3], at::kBFloat16, &Wm) || !matrix(*Wm, &wm) || wm.rows != w.rows || wm.cols != w.cols || wm.ld != w.ld))
    return declined();
  if (!stream_of(a[4], &s)) return declined();
  at::Tensor mask;
  const at::Device device = W->device();
  const uint16_t* wp = pointer<uint16_t>(W);
  uint16_t* wmp = pointer<uint16_t>(Wm);
  const int32_t st = unlocked([&] {
    mask = fresh(device, w.rows, (w.cols + 31) / 32, at::kInt);
    return lib.prune(wp, w.rows, w.cols, w.ld, N, M, pointer<uint32_t>(&mask), wmp, s);
  });
  return result(st, THPVariable_Wrap(std::move(mask)));
  END_HANDLE_TH_ERRORS
}

// prune_scored(score, N, M, stream)
PyObject* prune_scored(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor* score;
  Matrix m;
  int32_t N, M;
  void* s;
  if (n != 4 || observed() || !plain(a[0], at::kFloat, &score) || !matrix(*score, &m) || !level(a[1], a[2], &N, &M) ||
      !stream_of(a[3], &s))
    return declined();
  at::Tensor mask;
  const at::Device device = score->device();
  const float* sp = pointer<float>(score);
  const int32_t st = unlocked([&] {
    mask = fresh(device, m.rows, (m.cols + 31) / 32, at::kInt);
    return lib.prune_scored(sp, m.rows, m.cols, m.ld, N, M, pointer<uint32_t>(&mask), s);
  });
  return result(st, THPVariable_Wrap(std::move(mask)));
  END_HANDLE_TH_ERRORS
}

// pack(W, N, M, mask, stream)
PyObject* pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *W, *mask = nullptr;
  Matrix w;
  int32_t N, M;
  void* s;
  if (n != 5 || observed() || !plain(a[0], at::kBFloat16, &W) || !matrix(*W, &w) || w.rows < 1 || !level(a[1], a[2], &N, &M))
    return declined();
  if (a[3] != Py_None && (!plain(a[3], at::kInt, &mask) || !whole(*mask) || mask->size(0) != w.rows || mask->size(1) != (w.cols + 31) / 32))
    return declined();
  const size_t vb = lib.values_bytes(w.rows, w.cols, N, M);
  if (vb == 0 || !stream_of(a[4], &s)) return declined();
  at::Tensor values, indices;
  const at::Device device = W->device();
  const uint16_t* wp = pointer<uint16_t>(W);
  const uint32_t* mp = pointer<uint32_t>(mask);
  const int32_t st = unlocked([&] {
    values = fresh(device, w.rows, (int64_t)vb / (2 * w.rows), at::kBFloat16);
    indices = fresh(device, w.rows, (int64_t)lib.index_bytes(w.rows, w.cols, N, M) / (4 * w.rows), at::kInt);
    return lib.pack(wp, w.rows, w.cols, w.ld, N, M, mp, pointer<uint16_t>(&values), pointer<uint32_t>(&indices), s);
  });
  return result(st, Py_BuildValue("(NN)", THPVariable_Wrap(std::move(values)), THPVariable_Wrap(std::move(indices))));
  END_HANDLE_TH_ERRORS
}

// unpack(values, indices, K, N, M, stream)
PyObject* unpack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *values, *indices;
  int64_t K;
  int32_t N, M;
  void* s;
  if (n != 6 || observed() || !plain(a[0], at::kBFloat16, &values) || !whole(*values) || !plain(a[1], at::kInt, &indices) ||
      !whole(*indices) || !integer(a[2], 1, 1ll << 40, &K) || !level(a[3], a[4], &N, &M) || !stream_of(a[5], &s))
    return declined();
  const int64_t O = values->size(0);
  at::Tensor Wd;
  const at::Device device = values->device();
  const uint16_t* vp = pointer<uint16_t>(values);
  const uint32_t* ip = pointer<uint32_t>(indices);
  const int32_t st = unlocked([&] {
    Wd = fresh(device, O, K, at::kBFloat16);
    return lib.unpack(vp, ip, O, K, N, M, pointer<uint16_t>(&Wd), K, s);
  });
  return result(st, THPVariable_Wrap(std::move(Wd)));
  END_HANDLE_TH_ERRORS
}

// forward(values, indices, K, N, M, X, bias, out_dtype, out, workspace, stream, how); how: 0 plain, 1 prepared, 2 straight
// from the packed format, 3 on the library's fixed scratch
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *values, *indices, *X, *bias = nullptr, *out = nullptr, *ws = nullptr;
  int64_t K, how;
  int32_t N, M;
  Matrix x, y;
  void* s;
  if (n != 12 || observed() || !plain(a[0], at::kBFloat16, &values) || !whole(*values) || !plain(a[1], at::kInt, &indices) ||
      !whole(*indices) || !integer(a[2], 1, 1ll << 40, &K) || !level(a[3], a[4], &N, &M) || !plain(a[5], at::kBFloat16, &X) ||
      !matrix(*X, &x) || x.cols != K || !integer(a[11], 0, 3, &how))
    return declined();
  const int64_t O = values->size(0), T = x.rows;
  if (a[6] != Py_None && (!plain(a[6], at::kFloat, &bias) || bias->numel() != O || !bias->is_contiguous())) return declined();
  int32_t code;
  at::Tensor made;
  if (a[8] != Py_None) {
    if (plain(a[8], at::kBFloat16, &out)) code = NM_OUT_BF16;
    else if (plain(a[8], at::kFloat, &out)) code = NM_OUT_F32;
    else return declined();
    if (!matrix(*out, &y) || y.rows != T || y.cols != O) return declined();
  } else {
    at::ScalarType type = at::kFloat;
    if (a[7] != Py_None) {
      if (!THPDtype_Check(a[7])) return declined();
      type = reinterpret_cast<THPDtype*>(a[7])->scalar_type;
      if (type != at::kFloat && type != at::kBFloat16) return declined();
    }
    code = type == at::kFloat ? NM_OUT_F32 : NM_OUT_BF16;
  }
  if (!stream_of(a[10], &s)) return declined();
  THPObjectPtr found;  // a workspace looked up here, held until the call has returned
  void* ws_ptr = nullptr;
  size_t ws_bytes = 0;
  if (how != 3) {
    PyObject* given = a[9];
    if (given == Py_None && how != 2) {
      const size_t need = lib.workspace_bytes(O, K, N, M, T);
      if (need != 0 && how == 1) return declined();  // (refused, or a ragged reduction without its copy)
      if (need != 0) {
        PyObject* device = PyObject_GetAttrString(a[5], "device");
        if (device == nullptr) return nullptr;
        found = PyObject_CallFunction(find_workspace, "nNO", (Py_ssize_t)need, device, a[10]);
        if (!found) return nullptr;
        given = found.get();
      }
    }
    if (given != Py_None) {
      if (!THPVariable_CheckExact(given) || !(ws = &THPVariable_Unpack(given))->is_cuda() || !ws->has_storage()) {
        return declined();
      }
      ws_ptr = ws->data_ptr();
      ws_bytes = ws->nbytes();
    }
  }
  // partial sums of a prepared layer that is cut along K: scratch of the call, allocated on its stream, so that the memory goes to
  // later work of that stream only.  (Not for a workspace of the operand part alone, which asks for the uncut product.)
  size_t scratch_bytes = how == 1 && lib.prepared_scratch_bytes ? lib.prepared_scratch_bytes(O, K, N, M, T) : 0;
  if (scratch_bytes != 0 && ws_bytes < lib.workspace_bytes(O, K, N, M, T)) scratch_bytes = 0;
  at::Device here = X->device();
  if (scratch_bytes != 0) {
    here = at::Device(at::kCUDA, c10::hip::current_device());
    if (s != c10::hip::getCurrentHIPStream(here.index()).stream()) return declined();
  }
  const uint16_t *v = pointer<uint16_t>(values), *xp = pointer<uint16_t>(X);
  const uint32_t* ix = pointer<uint32_t>(indices);
  const float* b = pointer<float>(bias);
  void* yp = pointer<void>(out);
  const at::Device device = X->device();
  const int32_t st = unlocked([&] {
    if (out == nullptr) {
      made = fresh(device, T, O, code == NM_OUT_F32 ? at::kFloat : at::kBFloat16);
      yp = made.data_ptr();
      y.ld = O;
    }
    if (how == 3) return lib.forward_static(v, ix, O, K, N, M, xp, T, x.ld, b, yp, y.ld, code, s);
    if (scratch_bytes != 0) {
      const at::Tensor scratch = fresh(here, 1, (int64_t)scratch_bytes, at::kByte);
      return lib.forward_prepared_scratch(v, ix, O, K, N, M, xp, T, x.ld, b, yp, y.ld, code, ws_ptr, ws_bytes,
                                          scratch.data_ptr(), scratch_bytes, s);
    }
    if (how == 1) return lib.forward_prepared(v, ix, O, K, N, M, xp, T, x.ld, b, yp, y.ld, code, ws_ptr, ws_bytes, s);
    return lib.forward(v, ix, O, K, N, M, xp, T, x.ld, b, yp, y.ld, code, ws_ptr, ws_bytes, s);
  });
  if (out != nullptr) {
    Py_INCREF(a[8]);
    return result(st, a[8]);
  }
  return result(st, THPVariable_Wrap(std::move(made)));
  END_HANDLE_TH_ERRORS
}

// bind(addresses by name, raise_status, find_workspace)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *table, *raise, *find;
  if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &table, &raise, &find)) return nullptr;
  Library l = {};
  struct { const char* name; void* slot; bool optional = false; } slots[] = {
      {"nm_prune", &l.prune}, {"nm_prune_scored", &l.prune_scored}, {"nm_pack", &l.pack}, {"nm_unpack", &l.unpack},
      {"nm_linear_forward", &l.forward}, {"nm_linear_forward_prepared", &l.forward_prepared},
      {"nm_linear_forward_static", &l.forward_static}, {"nm_spmm_workspace_bytes", &l.workspace_bytes},
      {"nm_values_bytes", &l.values_bytes}, {"nm_index_bytes", &l.index_bytes},
      {"nm_linear_forward_prepared_scratch", &l.forward_prepared_scratch, true},
      {"nm_prepared_scratch_bytes", &l.prepared_scratch_bytes, true}};
  for (auto& e : slots) {
    PyObject* address = PyDict_GetItemString(table, e.name);
    if (address == nullptr && e.optional) continue;
    void* p = address ? PyLong_AsVoidPtr(address) : nullptr;
    if (p == nullptr) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "%s", e.name);
      return nullptr;
    }
    *static_cast<void**>(e.slot) = p;
  }
  lib = l;
  Py_INCREF(raise);
  Py_XSETREF(raise_status, raise);
  Py_INCREF(find);
  Py_XSETREF(find_workspace, find);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"prune", (PyCFunction)(void (*)())prune, METH_FASTCALL, nullptr},
    {"prune_scored", (PyCFunction)(void (*)())prune_scored, METH_FASTCALL, nullptr},
    {"pack", (PyCFunction)(void (*)())pack, METH_FASTCALL, nullptr},
    {"unpack", (PyCFunction)(void (*)())unpack, METH_FASTCALL, nullptr},
    {"forward", (PyCFunction)(void (*)())forward, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nm_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nm_calls() { return PyModule_Create(&module); }
