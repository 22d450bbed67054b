// CPython module between the Python entry points and the C ABI: the checks, the output allocation, the current
// stream and the call, for the arguments that a program passes in the usual case.  Anything else -- a wrong type, a
// wrong shape, a status other than RTOPK_OK -- makes the functions return None, and the Python code behind the same entry
// point then raises what it always raised (or makes the call without scratch memory, whose launch writes every output, should
// a launch of a split call have been refused).
//
// Why native: at the sizes of a sampled mini-batch the kernel takes 3 us and the Python form of these steps (ten
// attribute reads, two torch.empty, a stream lookup, a ctypes call of eight arguments) took 10 us.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/Context.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>

#include <exception>
#include <limits>

#include "rtopk.h"

namespace {

using at::Tensor;

// A tensor argument; nullptr where it is none.
const Tensor* tensor_of(PyObject* o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

// A whole number that fits 32 bits: a Python int, or whatever counts as an index (NumPy's integers).  What does not, or
// raises, is left to the Python code, with no exception set.
bool int32_of(PyObject* o, int32_t& v) {
  PyObject* made = nullptr;
  if (!PyLong_Check(o)) {
    if (!PyIndex_Check(o) || !(made = PyNumber_Index(o))) {
      PyErr_Clear();
      return false;
    }
    o = made;
  }
  int overflow = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
  Py_XDECREF(made);
  if (overflow != 0 || x < std::numeric_limits<int32_t>::min() || x > std::numeric_limits<int32_t>::max()) return false;
  v = (int32_t)x;
  return true;
}

// A number as a float: a Python float or int, or whatever converts to one.
bool float_of(PyObject* o, float& v) {
  const double x = PyFloat_Check(o) ? PyFloat_AS_DOUBLE(o) : (PyUnicode_Check(o) ? -1.0 : PyFloat_AsDouble(o));
  if (x == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  v = (float)x;
  return !PyUnicode_Check(o);
}

bool is_matrix(const Tensor& t, at::ScalarType type) {
  return t.is_cuda() && t.scalar_type() == type && t.dim() == 2 && t.is_contiguous();
}

bool is_shape(const Tensor& t, at::ScalarType type, int64_t rows, int64_t cols) {
  return is_matrix(t, type) && t.size(0) == rows && t.size(1) == cols;
}

// Whether a call is plain: no dispatch key beyond the default ones is switched on for the thread (modes, function transforms,
// tracing ...), no profiler listens, and new memory is not to be filled.
bool is_plain() {
  return (c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() && !at::hasCallbacks() &&
         !at::globalContext().deterministicAlgorithms();
}

// A new tensor on the device.  at::empty goes through the dispatcher twice, which is most of its 0.65 us; a plain call makes the
// tensor directly, by the same allocator (64 x 256, k = 32, two outputs, a call among others: 5.15 -> 4.70 us, the medians of four
// runs of either in turn, each within 0.05).
Tensor new_tensor(at::IntArrayRef shape, at::ScalarType type, c10::Device device, bool plain) {
  if (!plain) return at::empty(shape, at::TensorOptions().dtype(type).device(device));
  return Tensor(at::detail::empty_cuda(shape, type, device, std::nullopt));
}

// An output: the caller's, if it fits, or a new one.  `object` is a new reference to what the caller gets back.
struct Output {
  Tensor tensor;
  PyObject* object = nullptr;
  ~Output() { Py_XDECREF(object); }
  bool set(PyObject* given, at::ScalarType type, at::IntArrayRef shape, c10::Device device, bool plain) {
    if (given != Py_None) {
      const Tensor* t = tensor_of(given);
      if (!t || !t->is_cuda() || t->scalar_type() != type || !t->is_contiguous() || t->sizes() != shape) return false;
      tensor = *t;
      object = Py_NewRef(given);
      return true;
    }
    tensor = new_tensor(shape, type, device, plain);
    object = THPVariable_Wrap(tensor);
    return object != nullptr;
  }
  PyObject* release() {
    PyObject* o = object;
    object = nullptr;
    return o;
  }
};

void* stream_of(const Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// f() with C++ exceptions turned into Python's.  Without memory for an output the caller gets None, so that it makes the
// allocation itself and the user sees torch's own exception.
template <typename F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (const c10::OutOfMemoryError& e) {
    Py_RETURN_NONE;
  } catch (const std::exception& e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// call() without the interpreter lock.
template <typename F>
int unlocked(F call) {
  PyThreadState* state = PyEval_SaveThread();
  const int status = call();  // a C function: does not throw
  PyEval_RestoreThread(state);
  return status;
}

PyObject* none() { Py_RETURN_NONE; }

PyObject* pair(Output& a, Output& b) {
  PyObject* t = PyTuple_New(2);
  if (!t) return nullptr;
  PyTuple_SET_ITEM(t, 0, a.release());
  PyTuple_SET_ITEM(t, 1, b.release());
  return t;
}

// Scratch memory for a shape that can use it (rtopk_workspace_bytes), from torch's allocator: stream-ordered, so it may
// go back as soon as the call has enqueued its work on the current stream.  Where there is no memory for it the call does
// without.
struct Scratch {
  Tensor tensor;
  void* data = nullptr;
  int64_t bytes = 0;
  Scratch(const Tensor& x, int32_t k, int32_t variant, int32_t max_iter, bool plain) {
    bytes = rtopk_workspace_bytes(x.size(0), (int32_t)x.size(1), k, variant, max_iter);
    if (bytes > 0) {
      try {
        tensor = new_tensor({bytes}, at::kByte, x.device(), plain);
        data = tensor.data_ptr();
      } catch (const c10::OutOfMemoryError&) {
        bytes = 0;
      }
    }
  }
};

// select(which, x, k, max_iter, out_vals, out_idx): the entry points that return pairs.  which: 0 fp32, 1 fp32 with
// byte-wide columns, 2 the k smallest, 3 half, 4 bfloat16; plus 8 for exact mode (max_iter is then not looked at).
PyObject* select(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int32_t which, k, max_iter;
    if (n != 6 || !int32_of(args[0], which) || !int32_of(args[2], k) || !int32_of(args[3], max_iter) || k < 0) return none();
    const bool exact = (which & 8) != 0;
    which &= 7;
    const Tensor* x = tensor_of(args[1]);
    const at::ScalarType vt = which == 3 ? at::kHalf : (which == 4 ? at::kBFloat16 : at::kFloat);
    const at::ScalarType it = which == 1 ? at::kByte : at::kInt;
    if (!x || !is_matrix(*x, vt)) return none();
    const int64_t N = x->size(0), M = x->size(1);
    if (M > std::numeric_limits<int32_t>::max()) return none();
    const bool plain = is_plain();
    Output v, i;
    if (!v.set(args[4], vt, {N, k}, x->device(), plain) || !i.set(args[5], it, {N, k}, x->device(), plain))
      return PyErr_Occurred() ? nullptr : none();
    const void* in = x->data_ptr();
    void *ov = v.tensor.data_ptr(), *oi = i.tensor.data_ptr(), *s = stream_of(*x);
    const int32_t m = (int32_t)M;
    const int32_t variant = (exact ? RTOPK_EXACT : RTOPK_EARLY) + (which == 2 ? RTOPK_SMALLEST : 0);
    Scratch w(*x, which == 0 || which == 2 ? k : 0, variant, max_iter, plain);  // (none for k = 0)
    const int status = unlocked([&]() -> int {
      if (w.bytes > 0)
        return rtopk_select_ws(static_cast<const float*>(in), N, m, k, variant, max_iter, 0.0f, static_cast<float*>(ov),
                               static_cast<int32_t*>(oi), nullptr, w.data, w.bytes, s);
      const float* f = static_cast<const float*>(in);
      const uint16_t* h = static_cast<const uint16_t*>(in);
      float* fv = static_cast<float*>(ov);
      uint16_t* hv = static_cast<uint16_t*>(ov);
      int32_t* ii = static_cast<int32_t*>(oi);
      uint8_t* bi = static_cast<uint8_t*>(oi);
      switch (which) {
        case 0: return exact ? rtopk_rowwise_exact(f, N, m, k, fv, ii, s) : rtopk_rowwise(f, N, m, k, max_iter, fv, ii, s);
        case 1: return exact ? rtopk_rowwise_exact_u8(f, N, m, k, fv, bi, s) : rtopk_rowwise_u8(f, N, m, k, max_iter, fv, bi, s);
        case 2: return exact ? rtopk_rowwise_exact_smallest(f, N, m, k, fv, ii, s) : rtopk_rowwise_smallest(f, N, m, k, max_iter, fv, ii, s);
        case 3: return exact ? rtopk_rowwise_exact_f16(h, N, m, k, hv, ii, s) : rtopk_rowwise_f16(h, N, m, k, max_iter, hv, ii, s);
        case 4: return exact ? rtopk_rowwise_exact_bf16(h, N, m, k, hv, ii, s) : rtopk_rowwise_bf16(h, N, m, k, max_iter, hv, ii, s);
        default: return RTOPK_ERR_BAD_SHAPE;
      }
    });
    return status == RTOPK_OK ? pair(v, i) : none();
  });
}

// select_eps(x, k, eps_rel, out_vals, out_idx, out_iters, want_iters)
PyObject* select_eps(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int32_t k;
    float eps;
    if (n != 7 || !int32_of(args[1], k) || k < 0 || !float_of(args[2], eps)) return none();
    const int iters = args[5] != Py_None ? 1 : PyObject_IsTrue(args[6]);
    if (iters < 0) return nullptr;
    const Tensor* x = tensor_of(args[0]);
    if (!x || !is_matrix(*x, at::kFloat)) return none();
    const int64_t N = x->size(0), M = x->size(1);
    if (M > std::numeric_limits<int32_t>::max()) return none();
    const bool plain = is_plain();
    Output v, i, t;
    if (!v.set(args[3], at::kFloat, {N, k}, x->device(), plain) || !i.set(args[4], at::kInt, {N, k}, x->device(), plain) ||
        (iters != 0 && !t.set(args[5], at::kInt, {N}, x->device(), plain)))
      return PyErr_Occurred() ? nullptr : none();
    const float* in = static_cast<const float*>(x->data_ptr());
    float* ov = static_cast<float*>(v.tensor.data_ptr());
    int32_t* oi = static_cast<int32_t*>(i.tensor.data_ptr());
    int32_t* ot = iters != 0 ? static_cast<int32_t*>(t.tensor.data_ptr()) : nullptr;
    void* s = stream_of(*x);
    Scratch w(*x, k, RTOPK_EPS, 0, plain);
    const int status = unlocked([&] {
      return rtopk_select_ws(in, N, (int32_t)M, k, RTOPK_EPS, 0, eps, ov, oi, ot, w.data, w.bytes, s);
    });
    if (status != RTOPK_OK) return none();
    if (iters == 0) return pair(v, i);
    PyObject* r = PyTuple_New(3);
    if (!r) return nullptr;
    PyTuple_SET_ITEM(r, 0, v.release());
    PyTuple_SET_ITEM(r, 1, i.release());
    PyTuple_SET_ITEM(r, 2, t.release());
    return r;
  });
}

// dense(x, k, max_iter, out)
PyObject* dense(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int32_t k, max_iter;
    if (n != 4 || !int32_of(args[1], k) || !int32_of(args[2], max_iter)) return none();
    const Tensor* x = tensor_of(args[0]);
    if (!x || !is_matrix(*x, at::kFloat)) return none();
    const int64_t N = x->size(0), M = x->size(1);
    if (M > std::numeric_limits<int32_t>::max()) return none();
    const bool plain = is_plain();
    Output y;
    if (!y.set(args[3], at::kFloat, {N, M}, x->device(), plain)) return PyErr_Occurred() ? nullptr : none();
    const float* in = static_cast<const float*>(x->data_ptr());
    float* out = static_cast<float*>(y.tensor.data_ptr());
    void* s = stream_of(*x);
    const int status = unlocked([&] { return rtopk_maxk_dense(in, N, (int32_t)M, k, max_iter, out, s); });
    return status == RTOPK_OK ? y.release() : none();
  });
}

// scatter(grad_vals, idx, M, grad_in) and gather(grad_out, idx, grad_vals)
PyObject* scatter(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int32_t M;
    if (n != 4 || !int32_of(args[2], M) || M < 0) return none();
    const Tensor *g = tensor_of(args[0]), *idx = tensor_of(args[1]);
    if (!g || !idx) return none();
    const bool u8 = idx->scalar_type() == at::kByte;
    if (!is_matrix(*idx, u8 ? at::kByte : at::kInt) || (u8 && M > 256)) return none();
    const int64_t N = idx->size(0), k = idx->size(1);
    if (k > std::numeric_limits<int32_t>::max() || !is_shape(*g, at::kFloat, N, k)) return none();
    const bool plain = is_plain();
    Output y;
    if (!y.set(args[3], at::kFloat, {N, M}, idx->device(), plain)) return PyErr_Occurred() ? nullptr : none();
    const float* gv = static_cast<const float*>(g->data_ptr());
    const void* ix = idx->data_ptr();
    float* out = static_cast<float*>(y.tensor.data_ptr());
    void* s = stream_of(*idx);
    const int status = unlocked([&] {
      return u8 ? rtopk_maxk_backward_u8(gv, static_cast<const uint8_t*>(ix), N, M, (int32_t)k, out, s)
                : rtopk_maxk_backward(gv, static_cast<const int32_t*>(ix), N, M, (int32_t)k, out, s);
    });
    return status == RTOPK_OK ? y.release() : none();
  });
}

PyObject* gather(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 3) return none();
    const Tensor *g = tensor_of(args[0]), *idx = tensor_of(args[1]);
    if (!g || !idx || !is_matrix(*g, at::kFloat)) return none();
    const int64_t N = g->size(0), M = g->size(1);
    const bool u8 = idx->scalar_type() == at::kByte;
    if (!is_matrix(*idx, u8 ? at::kByte : at::kInt) || (u8 && M > 256) || idx->size(0) != N) return none();
    const int64_t k = idx->size(1);
    if (k > std::numeric_limits<int32_t>::max() || M > std::numeric_limits<int32_t>::max()) return none();
    const bool plain = is_plain();
    Output y;
    if (!y.set(args[2], at::kFloat, {N, k}, idx->device(), plain)) return PyErr_Occurred() ? nullptr : none();
    const float* go = static_cast<const float*>(g->data_ptr());
    const void* ix = idx->data_ptr();
    float* out = static_cast<float*>(y.tensor.data_ptr());
    void* s = stream_of(*idx);
    const int status = unlocked([&] {
      return u8 ? rtopk_maxk_backward_gather_u8(go, static_cast<const uint8_t*>(ix), N, (int32_t)M, (int32_t)k, out, s)
                : rtopk_maxk_backward_gather(go, static_cast<const int32_t*>(ix), N, (int32_t)M, (int32_t)k, out, s);
    });
    return status == RTOPK_OK ? y.release() : none();
  });
}

template <typename F>
PyCFunction fast(F f) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef kMethods[] = {
    {"select", fast(select), METH_FASTCALL, nullptr},   {"select_eps", fast(select_eps), METH_FASTCALL, nullptr},
    {"dense", fast(dense), METH_FASTCALL, nullptr},     {"scatter", fast(scatter), METH_FASTCALL, nullptr},
    {"gather", fast(gather), METH_FASTCALL, nullptr},   {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_rtopk_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rtopk_torch(void) { return PyModule_Create(&kModule); }
