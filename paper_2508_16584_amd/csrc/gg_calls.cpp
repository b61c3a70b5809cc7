// The everyday form of the binding's calls in native code: fresh outputs, the current stream, the automatic choice.
//
// A small call is bound by the host.  4 groups of 88 rows on average, N = K = 256, calls one after the other: 9.6 us with the
// checks, the allocation and the marshalling in Python, 4 of them the library's (most of it the launch); 5.5 here.  The seven calls
// of a small layer's forward and backward pass (64 tokens): 65.8 -> 48.4 us, of which the GPU now works nearly all.
// A function takes only what is plainly right - tensors of exactly torch's type, shapes, types and devices as the library
// wants them, no mode or transform at work - and returns None otherwise, without having launched anything: the binding's
// own code then takes the call, or says what is wrong with it.  The same when the library refuses the arguments.  An error of the
// HIP runtime, after which a launch may or may not be queued, is raised at once: the call is never made twice.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include <pthread.h>

#include "gg_fp8.h"

namespace {

// the library's functions, by the addresses that the binding found in the library it loaded
struct Library {
  decltype(&gg_fp8_grouped_gemm_ex) gemm;
  decltype(&gg_fp8_grouped_gemm_swiglu) gemm_swiglu;
  decltype(&gg_fp8_grouped_gemm_wgrad_ex) wgrad;
  decltype(&gg_fp8_quantize_rows_ex) quantize_rows;
  decltype(&gg_fp8_quantize_cols) quantize_cols;
  decltype(&gg_fp8_swiglu_quantize_rows_ex) swiglu_quantize_rows;
  decltype(&gg_fp8_swiglu_route) swiglu_route;      // null: always the fused call
} lib;
PyObject* check;      // the binding's function that raises the exception of a status

// a contiguous tensor of this type in device memory, and nothing that stands for one
const at::Tensor* plain(PyObject* o, at::ScalarType type, int64_t dim) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  static const c10::DispatchKeySet odd({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                        c10::DispatchKey::Functionalize, c10::DispatchKey::Batched, c10::DispatchKey::Conjugate,
                                        c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
  if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.dim() != dim || t.layout() != at::kStrided || t.key_set().has_any(odd) ||
      !t.has_storage() || !t.is_contiguous())
    return nullptr;
  return &t;
}

// a mode, a transform or a trace that would see the binding's own torch calls
bool seen_by_others() {
  static const c10::DispatchKeySet modes({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::PythonDispatcher,
                                          c10::DispatchKey::FuncTorchDynamicLayerFrontMode, c10::DispatchKey::FuncTorchDynamicLayerBackMode,
                                          c10::DispatchKey::FuncTorchVmapMode, c10::DispatchKey::VmapMode, c10::DispatchKey::Functionalize,
                                          c10::DispatchKey::Tracer});
  return c10::impl::tls_local_dispatch_key_set().included_.has_any(modes) || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
         at::impl::torch_function_mode_enabled();
}

bool fits(const at::Tensor* t, int64_t a, int64_t b) { return t->size(0) == a && t->size(1) == b; }
bool fits(const at::Tensor* t, int64_t a, int64_t b, int64_t c) { return t->size(0) == a && t->size(1) == b && t->size(2) == c; }
int64_t blocks(int64_t n) { return (n + 127) / 128; }
// exactly True or False: the truth of anything else is Python's to find
bool flag(PyObject* o, bool& value) {
  value = o == Py_True;
  return value || o == Py_False;
}
bool is_int(int64_t n) { return n <= 0x7FFFFFFF; }

// Without the interpreter's lock, as torch.empty allocates: an allocation can wait for the GPU.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor* like) {
  Unlocked unlocked;
  return at::empty(shape, at::TensorOptions().dtype(type).device(like->device()));
}
// the current stream of the current device, as the binding takes it
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

struct Gemm {
  const at::Tensor *A, *SA, *B, *SB, *off;
  int64_t G, M, N, K;
  // args: A, SA, B, SB, group_offsets
  bool read(PyObject* const* args, bool km) {
    A = plain(args[0], at::kByte, 2);
    SA = A ? plain(args[1], at::kFloat, 2) : nullptr;
    B = SA ? plain(args[2], at::kByte, 3) : nullptr;
    SB = B ? plain(args[3], at::kFloat, 3) : nullptr;
    off = SB ? plain(args[4], at::kInt, 1) : nullptr;
    if (!off) return false;
    M = A->size(0), K = A->size(1), G = B->size(0), N = B->size(1);
    return is_int(G) && is_int(N) && is_int(K) && B->size(2) == K && off->size(0) == G + 1 &&
           (km ? fits(SA, blocks(K), M) : fits(SA, M, blocks(K))) && fits(SB, G, blocks(N), blocks(K));
  }
};

// The library's call without the interpreter's lock, as ctypes makes it: a launch can wait for room in the stream's queue.
// False with an exception set: an error of the HIP runtime; without: the library refused the arguments.
template <class F, class... Args>
bool call(F* f, Args... args) {
  int status;
  Py_BEGIN_ALLOW_THREADS;
  status = f(args...);
  Py_END_ALLOW_THREADS;
  if (status == GG_ERR_HIP) Py_XDECREF(PyObject_CallFunction(check, "i", status));
  return status == GG_OK;
}

template <class T>
T* data(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }
template <class T>
T* data(const at::Tensor* t) { return static_cast<T*>(t->data_ptr()); }

PyObject* pair(const at::Tensor& a, const at::Tensor& b, const at::Tensor* c = nullptr, bool three = false) {
  PyObject* r = PyTuple_New(three ? 3 : 2);
  if (!r) return nullptr;
  PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(a));
  PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(b));
  if (three) {
    if (!c) Py_INCREF(Py_None);
    PyTuple_SET_ITEM(r, 2, c ? THPVariable_Wrap(*c) : Py_None);
  }
  return r;
}

// Every function: positional arguments only; no C++ exception leaves it (an allocation that fails is left to the binding's
// own code, which raises what torch raises).
template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    if (lib.gemm && !seen_by_others()) {
      PyObject* r = f();
      if (r || PyErr_Occurred()) return r;
    }
  } catch (...) {
  }
  Py_RETURN_NONE;
}

// (A, SA, B, SB, group_offsets, f16, sa_kmajor) -> C
PyObject* grouped_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    bool f16, km;
    Gemm g;
    if (!flag(args[5], f16) || !flag(args[6], km) || !g.read(args, km)) return nullptr;
    at::Tensor C = fresh({g.M, g.N}, f16 ? at::kHalf : at::kBFloat16, g.A);
    if (!call(lib.gemm, g.A->data_ptr(), data<float>(g.SA), g.B->data_ptr(), data<float>(g.SB), data<int32_t>(g.off), C.data_ptr(), (int)g.G, g.M, (int)g.N,
                 (int)g.K, nullptr, 0, current_stream(), -1, (km ? GG_SA_KMAJOR : 0) | (f16 ? GG_OUT_F16 : 0)))
      return nullptr;
    return THPVariable_Wrap(C);
  });
}

// (A, SA, B, SB, group_offsets, want_act, sa_kmajor) -> A2, SA2, act or None
PyObject* grouped_gemm_swiglu(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    bool want_act, km;
    Gemm g;
    if (!flag(args[5], want_act) || !flag(args[6], km) || !g.read(args, km) || g.N % 2) return nullptr;
    const int64_t inter = g.N / 2;
    at::Tensor A2 = fresh({g.M, inter}, at::kByte, g.A), act;
    at::Tensor SA2 = km ? fresh({inter / 128, g.M}, at::kFloat, g.A) : fresh({g.M, inter / 128}, at::kFloat, g.A);
    if (want_act) act = fresh({g.M, inter}, at::kBFloat16, g.A);
    const unsigned order = km ? GG_SA_KMAJOR : 0;
    if (lib.swiglu_route && lib.swiglu_route((int)g.G, g.M, (int)inter, (int)g.K, order) == 1) {
      // two launches, one after the other on the current stream, which is the intermediate's own; where memory has no room for it, one
      at::Tensor H;
      try {
        H = fresh({g.M, g.N}, at::kBFloat16, g.A);
      } catch (const c10::OutOfMemoryError&) {
      }
      if (H.defined()) {
        if (!call(lib.gemm, g.A->data_ptr(), data<float>(g.SA), g.B->data_ptr(), data<float>(g.SB), data<int32_t>(g.off), H.data_ptr(), (int)g.G, g.M, (int)g.N,
                  (int)g.K, nullptr, 0, current_stream(), -1, order) ||
            !call(lib.swiglu_quantize_rows, H.data_ptr(), A2.data_ptr(), data<float>(SA2), want_act ? act.data_ptr() : nullptr, g.M, (int)inter,
                  current_stream(), order))
          return nullptr;
        return pair(A2, SA2, want_act ? &act : nullptr, true);
      }
    }
    if (!call(lib.gemm_swiglu, g.A->data_ptr(), data<float>(g.SA), g.B->data_ptr(), data<float>(g.SB), data<int32_t>(g.off), A2.data_ptr(), data<float>(SA2),
                        want_act ? act.data_ptr() : nullptr, (int)g.G, g.M, (int)inter, (int)g.K, current_stream(), -1, order))
      return nullptr;
    return pair(A2, SA2, want_act ? &act : nullptr, true);
  });
}

// (XT, SX, DYT, SDY, group_offsets, out_bf16) -> dW
PyObject* grouped_gemm_wgrad(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 6, [&]() -> PyObject* {
    bool bf16;
    if (!flag(args[5], bf16)) return nullptr;
    const at::Tensor* XT = plain(args[0], at::kByte, 2);
    const at::Tensor* SX = XT ? plain(args[1], at::kFloat, 2) : nullptr;
    const at::Tensor* DYT = SX ? plain(args[2], at::kByte, 2) : nullptr;
    const at::Tensor* SDY = DYT ? plain(args[3], at::kFloat, 2) : nullptr;
    const at::Tensor* off = SDY ? plain(args[4], at::kInt, 1) : nullptr;
    if (!off) return nullptr;
    const int64_t K = XT->size(0), M = XT->size(1), N = DYT->size(0), G = off->size(0) - 1;
    if (G < 0 || !is_int(G) || !is_int(N) || !is_int(K) || DYT->size(1) != M || !fits(SX, blocks(M), K) || !fits(SDY, blocks(M), N)) return nullptr;
    at::Tensor dW = fresh({G, N, K}, bf16 ? at::kBFloat16 : at::kFloat, XT);
    if (!call(lib.wgrad, XT->data_ptr(), data<float>(SX), DYT->data_ptr(), data<float>(SDY), data<int32_t>(off), dW.data_ptr(), (int)G, M, (int)N, (int)K,
                  current_stream(), bf16 ? GG_OUT_BF16 : 0))
      return nullptr;
    return THPVariable_Wrap(dW);
  });
}

// X, row_src or None: the rows of the output
bool rows_of(PyObject* const* args, const at::Tensor*& X, const at::Tensor*& src, int64_t& M) {
  X = plain(args[0], at::kBFloat16, 2);
  if (!X || !is_int(X->size(1))) return false;
  src = nullptr;
  M = X->size(0);
  if (args[1] == Py_None) return true;
  src = plain(args[1], at::kInt, 1);
  if (src) M = src->size(0);
  return src != nullptr;
}

// (X, row_src, sa_kmajor) -> A, SA
PyObject* quantize_rows(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    const at::Tensor *X, *src;
    int64_t M;
    bool km;
    if (!flag(args[2], km) || !rows_of(args, X, src, M)) return nullptr;
    const int64_t T = X->size(0), K = X->size(1);
    at::Tensor A = fresh({M, K}, at::kByte, X);
    at::Tensor SA = km ? fresh({K / 128, M}, at::kFloat, X) : fresh({M, K / 128}, at::kFloat, X);
    if (!call(lib.quantize_rows, X->data_ptr(), src ? data<int32_t>(src) : nullptr, A.data_ptr(), data<float>(SA), T, M, (int)K, current_stream(),
                          km ? GG_SA_KMAJOR : 0))
      return nullptr;
    return pair(A, SA);
  });
}

// (X, row_src) -> XT, SX
PyObject* quantize_cols(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 2, [&]() -> PyObject* {
    const at::Tensor *X, *src;
    int64_t M;
    if (!rows_of(args, X, src, M)) return nullptr;
    const int64_t T = X->size(0), K = X->size(1);
    at::Tensor XT = fresh({K, M}, at::kByte, X), SX = fresh({blocks(M), K}, at::kFloat, X);
    if (!call(lib.quantize_cols, X->data_ptr(), src ? data<int32_t>(src) : nullptr, XT.data_ptr(), data<float>(SX), T, M, (int)K, current_stream()))
      return nullptr;
    return pair(XT, SX);
  });
}

// (H, want_act, sa_kmajor) -> A, SA, act or None
PyObject* swiglu_quantize_rows(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    const at::Tensor* H = plain(args[0], at::kBFloat16, 2);
    bool want_act, km;
    if (!H || H->size(1) % 2 || !is_int(H->size(1)) || !flag(args[1], want_act) || !flag(args[2], km)) return nullptr;
    const int64_t M = H->size(0), inter = H->size(1) / 2;
    at::Tensor A = fresh({M, inter}, at::kByte, H), act;
    at::Tensor SA = km ? fresh({inter / 128, M}, at::kFloat, H) : fresh({M, inter / 128}, at::kFloat, H);
    if (want_act) act = fresh({M, inter}, at::kBFloat16, H);
    if (!call(lib.swiglu_quantize_rows, H->data_ptr(), A.data_ptr(), data<float>(SA), want_act ? act.data_ptr() : nullptr, M, (int)inter, current_stream(),
                                 km ? GG_SA_KMAJOR : 0))
      return nullptr;
    return pair(A, SA, want_act ? &act : nullptr, true);
  });
}

// (addresses of the functions, in the order of Library, the last one may be missing; the function for `check`)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* p[7] = {};
  if (n < 7 || n > 8 || !PyCallable_Check(args[n - 1])) {
    PyErr_SetString(PyExc_TypeError, "six or seven addresses and a function");
    return nullptr;
  }
  for (int i = 0; i < n - 1; ++i) {
    p[i] = PyLong_AsVoidPtr(args[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  // A forked child may not use the GPU that its parent has used: torch says so, in the binding's own code.
  static const int forked = pthread_atfork(nullptr, nullptr, [] { lib = {}; });
  if (forked) Py_RETURN_NONE;
  Py_INCREF(args[n - 1]);
  Py_XSETREF(check, args[n - 1]);
  lib.gemm = reinterpret_cast<decltype(lib.gemm)>(p[0]);
  lib.gemm_swiglu = reinterpret_cast<decltype(lib.gemm_swiglu)>(p[1]);
  lib.wgrad = reinterpret_cast<decltype(lib.wgrad)>(p[2]);
  lib.quantize_rows = reinterpret_cast<decltype(lib.quantize_rows)>(p[3]);
  lib.quantize_cols = reinterpret_cast<decltype(lib.quantize_cols)>(p[4]);
  lib.swiglu_quantize_rows = reinterpret_cast<decltype(lib.swiglu_quantize_rows)>(p[5]);
  lib.swiglu_route = reinterpret_cast<decltype(lib.swiglu_route)>(p[6]);
  Py_RETURN_NONE;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(grouped_gemm), FAST(grouped_gemm_swiglu), FAST(grouped_gemm_wgrad), FAST(quantize_rows), FAST(quantize_cols),
                         FAST(swiglu_quantize_rows), FAST(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gg_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__gg_calls(void) { return PyModule_Create(&module); }
