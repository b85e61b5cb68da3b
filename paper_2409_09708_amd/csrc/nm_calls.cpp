// Native marshalling of the calls that a program makes per layer.  A small layer's call costs the host more than the device
// (one image through a 384 x 384 projection: 3.8 us of kernel, 7.3 us per call in Python), so a call whose arguments are all
// in the ordinary form -- plain device tensors of the right types and shapes, Python integers -- is read, checked and
// handed to the C ABI here.  Anything else is declined (NotImplemented), and the Python function goes on with it: it
// knows the other forms that are accepted and names what is wrong with the ones that are not.  Nothing is kept
// between calls.
// Measured per call: the projection above 7.3 -> 4.1 us; 768 -> 1000 at 4:8 on 8 tokens, plain, 8.2 -> 6.2 (5.0 with a kernel
// that has become faster since); the twelve calls and sixteen allocations that compress a block by scores and expand it 94 -> 63. The training
// products and the int8 layer on small operands: dX in one launch 7.2 -> 4.0 us (in two, with scratch of the call's own, 7.5 to 8.0), dW
// in two launches 11 -> 8, a prepared int8 call 7.5 -> 3.6; a plain call, whose scratch is looked up in the table that Python keeps,
// 4.0 -> 3.5.  (A launch alone takes the host 3.0 to 3.5; all of these vary by a quarter from host to host.)
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
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
  // may be missing: those calls are then declined
  decltype(&nm_linear_backward_input) backward_input;
  decltype(&nm_linear_backward_weight) backward_weight;
  decltype(&nm_linear_backward_input_scratch) backward_input_scratch;
  decltype(&nm_backward_input_workspace_bytes) backward_input_bytes;
  decltype(&nm_backward_input_scratch_bytes) backward_input_scratch_bytes;
  decltype(&nm_backward_input_scratch_pays) backward_input_scratch_pays;
  decltype(&nm_linear_backward_weight_scratch) backward_weight_scratch;
  decltype(&nm_backward_weight_scratch_bytes) backward_weight_scratch_bytes;
  decltype(&nm_linear_forward_i8) i8;
  decltype(&nm_linear_forward_i8_prepared) i8_prepared;
  decltype(&nm_linear_forward_i8_packed) i8_packed;
  decltype(&nm_linear_forward_i8_packed_prepared) i8_packed_prepared;
  decltype(&nm_i8_workspace_bytes) i8_bytes;
} lib;
PyObject* raise_status;    // raises NmError for a status that is not NM_OK
PyObject* find_workspace;  // the scratch tensor of a device and stream
PyObject* workspaces;      // where find_workspace keeps them: (device type, index, stream) -> tensor; may be missing

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

// Bytes that go to later work of this stream only, and back to it when the call has been issued.  Taken from the allocator without a
// tensor around them.
struct Scratch {
  void* ptr;
  Scratch(void* s, at::Device device, size_t bytes) {
    const c10::DeviceIndex current = c10::hip::current_device();
    c10::OptionalDeviceGuard on;
    if (device.index() != current && s != c10::hip::getCurrentHIPStream(current).stream()) on.reset_device(device);
    ptr = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, static_cast<hipStream_t>(s));
  }
  Scratch(const Scratch&) = delete;
  ~Scratch() { c10::hip::HIPCachingAllocator::raw_delete(ptr); }
};

// Whether memory allocated now, on the current device, goes to later work of this stream only.
bool on_current_stream(void* s, at::Device* here) {
  *here = at::Device(at::kCUDA, c10::hip::current_device());
  return s == c10::hip::getCurrentHIPStream(here->index()).stream();
}

// The workspace of a call: the given tensor, or the scratch of its device and stream, held until the call has returned.
struct Workspace {
  THPObjectPtr found;
  void* ptr = nullptr;
  size_t bytes = 0;
};
enum Take { TAKEN, DECLINED, FAILED };
Take given_workspace(PyObject* given, Workspace* w) {
  if (given == Py_None) return TAKEN;
  const at::Tensor* ws = nullptr;
  if (!THPVariable_CheckExact(given) || !(ws = &THPVariable_Unpack(given))->is_cuda() || !ws->has_storage()) return DECLINED;
  w->ptr = ws->data_ptr();
  w->bytes = ws->nbytes();
  return TAKEN;
}
// `like`: the tensor on whose device it lies (asking Python for it takes 0.7 us, reading its table 0.1)
Take scratch_workspace(size_t need, PyObject* like, PyObject* stream, void* s, Workspace* w) {
  if (workspaces != nullptr) {
    THPObjectPtr key(Py_BuildValue("(snK)", "cuda", (Py_ssize_t)THPVariable_Unpack(like).device().index(), (unsigned long long)(uintptr_t)s));
    if (!key) return FAILED;
    PyObject* kept = PyDict_GetItemWithError(workspaces, key.get());
    if (kept == nullptr && PyErr_Occurred()) return FAILED;
    if (kept != nullptr) {
      Py_INCREF(kept);
      w->found = THPObjectPtr(kept);
      if (given_workspace(kept, w) == TAKEN && w->bytes >= need) return TAKEN;
    }
  }
  THPObjectPtr device(PyObject_GetAttrString(like, "device"));
  if (!device) return FAILED;
  w->found = THPObjectPtr(PyObject_CallFunction(find_workspace, "nOO", (Py_ssize_t)need, device.get(), stream));
  return w->found ? given_workspace(w->found.get(), w) : FAILED;
}

// The output of a call: `given` (out), or made on the device of its operands in the type asked for (out_dtype).
struct Output {
  PyObject* given;
  at::Tensor made;
  at::ScalarType type;
  int64_t rows, cols, ld;
  void* ptr;
  int32_t code;
  bool read(PyObject* dtype, PyObject* out, int64_t r, int64_t c, bool i32) {
    given = out;
    rows = r;
    cols = c;
    type = at::kFloat;
    if (out != Py_None) {
      const at::Tensor* t = nullptr;
      Matrix m;
      if (!plain(out, at::kBFloat16, &t) && !plain(out, at::kFloat, &t) && !(i32 && plain(out, at::kInt, &t))) return false;
      if (!matrix(*t, &m) || m.rows != r || m.cols != c) return false;
      type = t->scalar_type();
      ld = m.ld;
      ptr = t->data_ptr();
    } else if (dtype != Py_None) {
      if (!THPDtype_Check(dtype)) return false;
      type = reinterpret_cast<THPDtype*>(dtype)->scalar_type;
    }
    if (type == at::kFloat) code = NM_OUT_F32;
    else if (type == at::kBFloat16) code = NM_OUT_BF16;
    else if (i32 && type == at::kInt) code = NM_OUT_I32;
    else return false;
    return true;
  }
  void make(at::Device device) {  // (without the interpreter lock)
    if (given != Py_None) return;
    made = fresh(device, rows, cols, type);
    ptr = made.data_ptr();
    ld = cols;
  }
  PyObject* take() {
    if (given == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
  }
};

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
  const at::Tensor *values, *indices, *X, *bias = nullptr, *out = nullptr;
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
  Workspace ws;
  if (how != 3) {
    if (a[9] == Py_None && how != 2) {
      const size_t need = lib.workspace_bytes(O, K, N, M, T);
      if (need != 0 && how == 1) return declined();  // (refused, or a ragged reduction without its copy)
      if (need != 0)
        if (const Take t = scratch_workspace(need, a[5], a[10], s, &ws); t != TAKEN) return t == DECLINED ? declined() : nullptr;
    } else if (given_workspace(a[9], &ws) != TAKEN) {
      return declined();
    }
  }
  void* const ws_ptr = ws.ptr;
  const size_t ws_bytes = ws.bytes;
  // partial sums of a prepared layer that is cut along K: scratch of the call, allocated on its stream, so that the memory goes to
  // later work of that stream only.  (Not for a workspace of the operand part alone, which asks for the uncut product.)
  size_t scratch_bytes = how == 1 && lib.prepared_scratch_bytes ? lib.prepared_scratch_bytes(O, K, N, M, T) : 0;
  if (scratch_bytes != 0 && ws_bytes < lib.workspace_bytes(O, K, N, M, T)) scratch_bytes = 0;
  at::Device here = X->device();
  if (scratch_bytes != 0 && !on_current_stream(s, &here)) return declined();
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

// backward_input(Ws, dY, out_dtype, out, workspace, stream)
PyObject* backward_input(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *W, *dY;
  Matrix w, dy;
  Output y;
  void* s;
  if (n != 6 || lib.backward_input == nullptr || lib.backward_input_scratch == nullptr || lib.backward_input_bytes == nullptr ||
      lib.backward_input_scratch_bytes == nullptr || lib.backward_input_scratch_pays == nullptr || observed() || !plain(a[0], at::kBFloat16, &W) ||
      !matrix(*W, &w) || !plain(a[1], at::kBFloat16, &dY) || !matrix(*dY, &dy) || dy.cols != w.rows ||
      !y.read(a[2], a[3], dy.rows, w.cols, false) || !stream_of(a[5], &s))
    return declined();
  Workspace ws;
  const size_t need = a[4] == Py_None ? lib.backward_input_bytes(w.rows, w.cols, dy.rows) : 0;
  if (const Take t = need != 0 ? scratch_workspace(need, a[1], a[5], s, &ws) : given_workspace(a[4], &ws); t != TAKEN)
    return t == DECLINED ? declined() : nullptr;
  // what a small layer can use: scratch of the call, as the partial sums above.  (A given workspace is left alone that is not required.)
  const size_t scratch_bytes = need == 0 && a[4] == Py_None && lib.backward_input_scratch_pays(w.rows, w.cols, dy.rows, y.code, s)
                                   ? lib.backward_input_scratch_bytes(w.rows, w.cols, dy.rows) : 0;
  const uint16_t *wp = pointer<uint16_t>(W), *dyp = pointer<uint16_t>(dY);
  const at::Device device = dY->device();
  const int32_t st = unlocked([&] {
    y.make(device);
    if (scratch_bytes != 0) {
      const Scratch scratch(s, device, scratch_bytes);
      return lib.backward_input_scratch(wp, w.rows, w.cols, w.ld, dyp, dy.rows, dy.ld, y.ptr, y.ld, y.code, scratch.ptr, scratch_bytes, s);
    }
    return lib.backward_input(wp, w.rows, w.cols, w.ld, dyp, dy.rows, dy.ld, y.ptr, y.ld, y.code, ws.ptr, ws.bytes, s);
  });
  return result(st, y.take());
  END_HANDLE_TH_ERRORS
}

// backward_weight(dY, X, mask, out_dtype, out, workspace, stream)
PyObject* backward_weight(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *dY, *X, *mask = nullptr;
  Matrix dy, x;
  Output y;
  void* s;
  if (n != 7 || lib.backward_weight == nullptr || lib.backward_weight_scratch == nullptr ||
      lib.backward_weight_scratch_bytes == nullptr || observed() || !plain(a[0], at::kBFloat16, &dY) ||
      !matrix(*dY, &dy) || !plain(a[1], at::kBFloat16, &X) || !matrix(*X, &x) || x.rows != dy.rows)
    return declined();
  if (a[2] != Py_None && (!plain(a[2], at::kInt, &mask) || !whole(*mask) || mask->size(0) != dy.cols || mask->size(1) != (x.cols + 31) / 32))
    return declined();
  if (!y.read(a[3], a[4], dy.cols, x.cols, false) || !stream_of(a[6], &s)) return declined();
  Workspace ws;
  const size_t need = a[5] == Py_None ? lib.backward_weight_scratch_bytes(dy.cols, x.cols, dy.rows) : 0;
  const auto call = a[5] == Py_None ? lib.backward_weight_scratch : lib.backward_weight;
  if (const Take t = need != 0 ? scratch_workspace(need, a[0], a[6], s, &ws) : given_workspace(a[5], &ws); t != TAKEN)
    return t == DECLINED ? declined() : nullptr;
  const uint16_t *dyp = pointer<uint16_t>(dY), *xp = pointer<uint16_t>(X);
  const uint32_t* mp = pointer<uint32_t>(mask);
  const at::Device device = dY->device();
  const int32_t st = unlocked([&] {
    y.make(device);
    return call(dyp, dy.rows, dy.cols, dy.ld, xp, x.cols, x.ld, mp, y.ptr, y.ld, y.code, ws.ptr, ws.bytes, s);
  });
  return result(st, y.take());
  END_HANDLE_TH_ERRORS
}

bool per_feature(PyObject* obj, int64_t O, const float** out) {
  const at::Tensor* t = nullptr;
  if (obj != Py_None && (!plain(obj, at::kFloat, &t) || t->numel() != O || !t->is_contiguous())) return false;
  *out = pointer<float>(t);
  return true;
}

// forward_i8(Wq, mask, None, N, M, Xq, x_scale, w_scale, bias, out_dtype, out, workspace, stream, prepared), or values, indices and K
// in the first three places
PyObject* forward_i8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *W, *words, *X;
  Matrix w, x;
  int64_t K, prepared;
  int32_t N, M;
  Output y;
  const float *scale, *bias;
  void* s;
  if (n != 14 || lib.i8_bytes == nullptr || observed() || !plain(a[0], at::kChar, &W) || !plain(a[1], at::kInt, &words) ||
      !whole(*words) || !matrix(*W, &w) || !level(a[3], a[4], &N, &M) || !plain(a[5], at::kChar, &X) || !matrix(*X, &x) ||
      !integer(a[13], 0, 1, &prepared))
    return declined();
  const bool packed = a[2] != Py_None;
  if (packed ? !W->is_contiguous() || !integer(a[2], 1, 1ll << 40, &K)
             : words->size(0) != w.rows || words->size(1) != ((K = w.cols) + 31) / 32)
    return declined();
  const int64_t O = w.rows, T = x.rows;
  if (x.cols != K || !per_feature(a[7], O, &scale) || !per_feature(a[8], O, &bias) || !y.read(a[9], a[10], T, O, true)) return declined();
  float x_scale;
  if (PyFloat_CheckExact(a[6])) x_scale = (float)PyFloat_AS_DOUBLE(a[6]);
  else return declined();
  if (!stream_of(a[12], &s)) return declined();
  Workspace ws;
  const size_t need = a[11] == Py_None ? lib.i8_bytes(O, K, N, M, T) : 0;
  if (need != 0 && prepared) return declined();  // (refused)
  if (const Take t = need != 0 ? scratch_workspace(need, a[5], a[12], s, &ws) : given_workspace(a[11], &ws); t != TAKEN)
    return t == DECLINED ? declined() : nullptr;
  const auto dense_call = prepared ? lib.i8_prepared : lib.i8;
  const auto packed_call = prepared ? lib.i8_packed_prepared : lib.i8_packed;
  if (packed ? packed_call == nullptr : dense_call == nullptr) return declined();
  const int8_t *wp = pointer<int8_t>(W), *xp = pointer<int8_t>(X);
  const uint32_t* mp = pointer<uint32_t>(words);
  const at::Device device = X->device();
  const int32_t st = unlocked([&] {
    y.make(device);
    if (packed) return packed_call(wp, mp, O, K, N, M, xp, T, x.ld, x_scale, scale, bias, y.ptr, y.ld, y.code, ws.ptr, ws.bytes, s);
    return dense_call(wp, O, K, w.ld, mp, N, M, xp, T, x.ld, x_scale, scale, bias, y.ptr, y.ld, y.code, ws.ptr, ws.bytes, s);
  });
  return result(st, y.take());
  END_HANDLE_TH_ERRORS
}

// bind(addresses by name, raise_status, find_workspace[, where that keeps its tensors])
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *table, *raise, *find, *kept = nullptr;
  if (!PyArg_ParseTuple(args, "O!OO|O!", &PyDict_Type, &table, &raise, &find, &PyDict_Type, &kept)) return nullptr;
  Library l = {};
  struct { const char* name; void* slot; bool optional = false; } slots[] = {
      {"nm_prune", &l.prune}, {"nm_prune_scored", &l.prune_scored}, {"nm_pack", &l.pack}, {"nm_unpack", &l.unpack},
      {"nm_linear_forward", &l.forward}, {"nm_linear_forward_prepared", &l.forward_prepared},
      {"nm_linear_forward_static", &l.forward_static}, {"nm_spmm_workspace_bytes", &l.workspace_bytes},
      {"nm_values_bytes", &l.values_bytes}, {"nm_index_bytes", &l.index_bytes},
      {"nm_linear_forward_prepared_scratch", &l.forward_prepared_scratch, true},
      {"nm_prepared_scratch_bytes", &l.prepared_scratch_bytes, true},
      {"nm_linear_backward_input", &l.backward_input, true}, {"nm_linear_backward_weight", &l.backward_weight, true},
      {"nm_linear_backward_input_scratch", &l.backward_input_scratch, true},
      {"nm_backward_input_workspace_bytes", &l.backward_input_bytes, true},
      {"nm_backward_input_scratch_bytes", &l.backward_input_scratch_bytes, true},
      {"nm_backward_input_scratch_pays", &l.backward_input_scratch_pays, true},
      {"nm_linear_backward_weight_scratch", &l.backward_weight_scratch, true},
      {"nm_backward_weight_scratch_bytes", &l.backward_weight_scratch_bytes, true}, {"nm_linear_forward_i8", &l.i8, true},
      {"nm_linear_forward_i8_prepared", &l.i8_prepared, true}, {"nm_linear_forward_i8_packed", &l.i8_packed, true},
      {"nm_linear_forward_i8_packed_prepared", &l.i8_packed_prepared, true}, {"nm_i8_workspace_bytes", &l.i8_bytes, true}};
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
  Py_XINCREF(kept);
  Py_XSETREF(workspaces, kept);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"prune", (PyCFunction)(void (*)())prune, METH_FASTCALL, nullptr},
    {"prune_scored", (PyCFunction)(void (*)())prune_scored, METH_FASTCALL, nullptr},
    {"pack", (PyCFunction)(void (*)())pack, METH_FASTCALL, nullptr},
    {"unpack", (PyCFunction)(void (*)())unpack, METH_FASTCALL, nullptr},
    {"forward", (PyCFunction)(void (*)())forward, METH_FASTCALL, nullptr},
    {"backward_input", (PyCFunction)(void (*)())backward_input, METH_FASTCALL, nullptr},
    {"backward_weight", (PyCFunction)(void (*)())backward_weight, METH_FASTCALL, nullptr},
    {"forward_i8", (PyCFunction)(void (*)())forward_i8, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nm_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nm_calls() { return PyModule_Create(&module); }
