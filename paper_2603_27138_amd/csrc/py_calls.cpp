// The library's entry points as Python functions that take torch tensors (CPython extension `_calls`).
//
// What a call costs the interpreter is what bounds a decode step of a few sequences: reading twenty
// arguments through ctypes (a Python call per tensor for its device, its layout and its address, and one
// for the current stream) took 17 us for scout_layer_step, while its launches take 6.  Here the tensors are
// looked into directly, and the C ABI is called through the addresses that the ctypes binding has loaded
// (bind), so there is one copy of the library.  Checks, messages and return codes are binding.py's: what is no plain
// tensor (subclasses, objects with a tensor's attributes, None where one is required) goes through its _ptr, and what
// torch throws becomes the Python exception that its own calls raise (entry).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/DeviceAccelerator.h>
#include <ATen/core/CachingHostAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "scout.h"

namespace {

// binding.py's Problem, _ptr, _ptr_addressable and _stream, filled by bind().
struct Binding {
  PyObject *problem = nullptr, *ptr = nullptr, *ptr_addressable = nullptr, *stream = nullptr;
} py;

// Calls one of them, which answers with a c_void_p or None; on an error the exception is set.
void* address_by(PyObject* f, PyObject* arg) {
  PyObject* const r = PyObject_CallFunctionObjArgs(f, arg, nullptr);
  PyObject* const value = r == nullptr || r == Py_None ? nullptr : PyObject_GetAttrString(r, "value");
  void* const address = value == nullptr || value == Py_None ? nullptr : PyLong_AsVoidPtr(value);
  Py_XDECREF(r);
  Py_XDECREF(value);
  return address;
}

// A pinned tensor that work on the current stream reads or writes: its memory goes to another tensor only after that work,
// however early the tensor itself is dropped.  (The allocator of pinned memory knows of copies by itself, of kernels it does not;
// memory that is not its own it leaves alone.)
void used_by_stream(const at::Tensor& t) {
  const at::DeviceType device = at::accelerator::getAccelerator(true).value();
  const at::DataPtr& memory = t.storage().data_ptr();
  at::getHostAllocator(device)->record_event(memory.get(), memory.get_context(),
                                             at::accelerator::getCurrentStream(at::accelerator::getDeviceIndex()));
}

// One argument list on its way to the C ABI: problem, tensors by position, then workspace and stream.
struct Args {
  const char* fn;
  PyObject* const* a;
  Py_ssize_t n, at = 0;
  bool ok = true;
  Py_buffer problem{};
  bool have_problem = false;

  Args(const char* fn_, PyObject* const* a_, Py_ssize_t n_, Py_ssize_t want) : fn(fn_), a(a_), n(n_) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "%s: %zd arguments expected, %zd given", fn, want, n);
      ok = false;
    }
  }
  ~Args() {
    if (have_problem) PyBuffer_Release(&problem);
  }
  Args(const Args&) = delete;
  Args& operator=(const Args&) = delete;

  PyObject* next() { return a[at++]; }

  const scout_problem* prob() {
    if (!ok) return nullptr;
    PyObject* const o = next();
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(py.problem))) {
      PyErr_Format(PyExc_TypeError, "%s: the first argument is a Problem, not %s", fn, Py_TYPE(o)->tp_name);
      ok = false;
      return nullptr;
    }
    if (PyObject_GetBuffer(o, &problem, PyBUF_SIMPLE) != 0) {
      ok = false;
      return nullptr;
    }
    have_problem = true;
    if (problem.len < (Py_ssize_t)sizeof(scout_problem)) {
      PyErr_Format(PyExc_TypeError, "%s: the Problem is too small", fn);
      ok = false;
    }
    return static_cast<const scout_problem*>(problem.buf);
  }

  // of an object that is no plain tensor: binding.py's answer
  void* by_python(PyObject* o, bool pinned) {
    void* const address = address_by(pinned ? py.ptr_addressable : py.ptr, o);
    if (PyErr_Occurred()) ok = false;
    return address;
  }

  // the address of a contiguous tensor; `pinned`: in device memory or in pinned host memory
  void* address(PyObject* o, bool pinned) {
    if (!THPVariable_CheckExact(o)) return by_python(o, pinned);
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_contiguous() || !(t.is_cuda() || (pinned && t.is_pinned()))) {
      PyErr_SetString(PyExc_AssertionError, pinned ? "need a CUDA tensor or a pinned CPU tensor"
                                                   : "device tensors must be contiguous CUDA tensors");
      ok = false;
      return nullptr;
    }
    if (!t.is_cuda()) used_by_stream(t);
    return t.data_ptr();
  }
  template <class T = void>
  T* dev() {  // None: a null pointer
    if (!ok) return nullptr;
    PyObject* const o = next();
    return o == Py_None ? nullptr : static_cast<T*>(address(o, false));
  }
  void* addressable() { return ok ? address(next(), true) : nullptr; }
  void* addressable_or_none() {
    if (!ok) return nullptr;
    PyObject* const o = next();
    return o == Py_None ? nullptr : address(o, true);
  }
  void* workspace(size_t* bytes) {
    *bytes = 0;
    if (!ok) return nullptr;
    PyObject* const o = next();
    void* const ws = address(o, false);
    if (!ok) return nullptr;
    if (THPVariable_CheckExact(o)) {
      *bytes = (size_t)THPVariable_Unpack(o).numel();
      return ws;
    }
    PyObject* const n = PyObject_CallMethod(o, "numel", nullptr);
    *bytes = n == nullptr ? 0 : (size_t)PyLong_AsUnsignedLongLongMask(n);
    Py_XDECREF(n);
    if (PyErr_Occurred()) ok = false;
    return ws;
  }
  int64_t integer() {
    if (!ok) return 0;
    PyObject* const as_int = PyNumber_Long(next());  // what int() takes
    const int64_t v = as_int ? (int64_t)PyLong_AsUnsignedLongLongMask(as_int) : -1;  // the low 64 bits, as ctypes passes them
    Py_XDECREF(as_int);
    if (v == -1 && PyErr_Occurred()) ok = false;
    return v;
  }
};

void* current_stream() {
  try {
    return c10::hip::getCurrentHIPStream().stream();
  } catch (const c10::Error&) {  // no usable device: what torch.cuda says of it
    return address_by(py.stream, nullptr);
  }
}

// Entry points by address, filled by bind().
struct Table {
  decltype(&::build_digests) build_digests;
  decltype(&::append_token) append_token;
  decltype(&::score_blocks) score_blocks;
  decltype(&::select_topk) select_topk;
  decltype(&::scout_select_ahead) scout_select_ahead;
  decltype(&::sparse_decode_attn) sparse_decode_attn;
  decltype(&::sparse_decode_attn_static) sparse_decode_attn_static;
  decltype(&::scout_attn_partials) scout_attn_partials;
  decltype(&::scout_attn_finish) scout_attn_finish;
  decltype(&::merge_partials) merge_partials;
  decltype(&::periodic_recall) periodic_recall;
  decltype(&::recall_fetch) recall_fetch;
  decltype(&::recall_scatter) recall_scatter;
  decltype(&::scout_layer_step) scout_layer_step;
} T;

// Every function returns the library's code; binding.py turns a negative one into ScoutError.
#define SCOUT_RETURN(CALL)                   \
  do {                                       \
    if (!A.ok) return nullptr;               \
    void* const st = current_stream();       \
    if (PyErr_Occurred()) return nullptr;    \
    int rc;                                  \
    Py_BEGIN_ALLOW_THREADS                   \
    rc = CALL;                               \
    Py_END_ALLOW_THREADS                     \
    return PyLong_FromLong(rc);              \
  } while (0)

typedef int32_t i32;

PyObject* py_build_digests(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("build_digests", a, n, 3);
  const auto* p = A.prob();
  void *k = A.dev(), *digest = A.dev();
  SCOUT_RETURN(T.build_digests(p, k, digest, st));
}

PyObject* py_append_token(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("append_token", a, n, 12);
  const auto* p = A.prob();
  i32* ctx = A.dev<i32>();
  void *k = A.dev(), *v = A.dev();
  i32* slot = A.dev<i32>();
  void* digest = A.dev();
  i32* table = A.dev<i32>();
  void *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  void *hk = A.addressable_or_none(), *hv = A.addressable_or_none();
  SCOUT_RETURN(T.append_token(p, ctx, k, v, slot, digest, table, kp, vp, slots, hk, hv, st));
}

PyObject* py_score_blocks(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("score_blocks", a, n, 5);
  const auto* p = A.prob();
  void *q = A.dev(), *digest = A.dev();
  float* scores = A.dev<float>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.score_blocks(p, q, digest, scores, ws, nws, st));
}

PyObject* py_select_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("select_topk", a, n, 10);
  const auto* p = A.prob();
  float* scores = A.dev<float>();
  i32 *table = A.dev<i32>(), *sel_all = A.dev<i32>(), *sel_gpu = A.dev<i32>(), *slot_gpu = A.dev<i32>(),
      *n_gpu = A.dev<i32>(), *sel_host = A.dev<i32>(), *n_host = A.dev<i32>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.select_topk(p, scores, table, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, ws, nws, st));
}

PyObject* py_select_ahead(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("scout_select_ahead", a, n, 14);
  const auto* p = A.prob();
  void *q = A.dev(), *digest = A.dev();
  i32* table = A.dev<i32>();
  float* scores = A.dev<float>();
  i32 *sel_all = A.dev<i32>(), *sel_gpu = A.dev<i32>(), *slot_gpu = A.dev<i32>(), *n_gpu = A.dev<i32>(),
      *sel_host = A.dev<i32>(), *n_host = A.dev<i32>();
  i32 *job_sel = static_cast<i32*>(A.addressable()), *job_n = static_cast<i32*>(A.addressable());
  void* job_q = A.addressable();
  SCOUT_RETURN(T.scout_select_ahead(p, q, digest, table, scores, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, job_sel,
                                    job_n, job_q, st));
}

PyObject* py_sparse_decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("sparse_decode_attn", a, n, 12);
  const auto* p = A.prob();
  void *q = A.dev(), *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  i32 *sel = A.dev<i32>(), *slot = A.dev<i32>(), *n_gpu = A.dev<i32>();
  float *o = A.dev<float>(), *m = A.dev<float>(), *l = A.dev<float>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.sparse_decode_attn(p, q, kp, vp, slots, sel, slot, n_gpu, o, m, l, ws, nws, st));
}

PyObject* py_sparse_decode_attn_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("sparse_decode_attn_static", a, n, 11);
  const auto* p = A.prob();
  void *q = A.dev(), *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  i32 *sel = A.dev<i32>(), *slot = A.dev<i32>(), *n_gpu = A.dev<i32>();
  float *o = A.dev<float>(), *m = A.dev<float>(), *l = A.dev<float>();
  SCOUT_RETURN(T.sparse_decode_attn_static(p, q, kp, vp, slots, sel, slot, n_gpu, o, m, l, st));
}

PyObject* py_attn_partials(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("scout_attn_partials", a, n, 9);
  const auto* p = A.prob();
  void *q = A.dev(), *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  i32 *sel = A.dev<i32>(), *slot = A.dev<i32>(), *n_gpu = A.dev<i32>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.scout_attn_partials(p, q, kp, vp, slots, sel, slot, n_gpu, ws, nws, st));
}

PyObject* py_attn_finish(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("scout_attn_finish", a, n, 7);
  const auto* p = A.prob();
  float *ho = A.dev<float>(), *hm = A.dev<float>(), *hl = A.dev<float>();
  void* out = A.dev();
  float* lse = A.dev<float>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.scout_attn_finish(p, ho, hm, hl, out, lse, ws, nws, st));
}

PyObject* py_attn_finish_ahead(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("scout_attn_finish", a, n, 7);
  const auto* p = A.prob();
  float *ho = static_cast<float*>(A.addressable()), *hm = static_cast<float*>(A.addressable()),
        *hl = static_cast<float*>(A.addressable());
  void* out = A.dev();
  float* lse = A.dev<float>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.scout_attn_finish(p, ho, hm, hl, out, lse, ws, nws, st));
}

PyObject* py_merge_partials(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("merge_partials", a, n, 9);
  const auto* p = A.prob();
  float *oa = A.dev<float>(), *ma = A.dev<float>(), *la = A.dev<float>();
  float *ob = A.dev<float>(), *mb = A.dev<float>(), *lb = A.dev<float>();
  void* out = A.dev();
  float* lse = A.dev<float>();
  SCOUT_RETURN(T.merge_partials(p, oa, ma, la, ob, mb, lb, out, lse, st));
}

PyObject* py_periodic_recall(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("periodic_recall", a, n, 9);
  const auto* p = A.prob();
  void *q = A.dev(), *digest = A.dev();
  i32 *table = A.dev<i32>(), *blk = A.dev<i32>(), *slot = A.dev<i32>(), *evict = A.dev<i32>(), *nr = A.dev<i32>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.periodic_recall(p, q, digest, table, blk, slot, evict, nr, ws, nws, st));
}

PyObject* py_recall_fetch(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("recall_fetch", a, n, 9);
  const auto* p = A.prob();
  void *sk = A.addressable(), *sv = A.addressable();
  i32 *blk = A.dev<i32>(), *slot = A.dev<i32>(), *nr = A.dev<i32>();
  void *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  SCOUT_RETURN(T.recall_fetch(p, sk, sv, blk, slot, nr, kp, vp, slots, st));
}

PyObject* py_recall_scatter(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("recall_scatter", a, n, 10);
  const auto* p = A.prob();
  void* staged = A.dev();
  const int64_t tiles = A.integer();
  i32 *off = A.dev<i32>(), *blk = A.dev<i32>(), *slot = A.dev<i32>(), *nr = A.dev<i32>();
  void *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  SCOUT_RETURN(T.recall_scatter(p, staged, tiles, off, blk, slot, nr, kp, vp, slots, st));
}

PyObject* py_layer_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args A("scout_layer_step", a, n, 20);
  const auto* p = A.prob();
  void *q = A.dev(), *digest = A.dev();
  i32* table = A.dev<i32>();
  void *kp = A.dev(), *vp = A.dev();
  const int64_t slots = A.integer();
  float *ho = A.dev<float>(), *hm = A.dev<float>(), *hl = A.dev<float>(), *scores = A.dev<float>();
  i32 *sel_all = A.dev<i32>(), *sel_gpu = A.dev<i32>(), *slot_gpu = A.dev<i32>(), *n_gpu = A.dev<i32>(),
      *sel_host = A.dev<i32>(), *n_host = A.dev<i32>();
  void* out = A.dev();
  float* lse = A.dev<float>();
  size_t nws;
  void* ws = A.workspace(&nws);
  SCOUT_RETURN(T.scout_layer_step(p, q, digest, table, kp, vp, slots, ho, hm, hl, scores, sel_all, sel_gpu, slot_gpu,
                                  n_gpu, sel_host, n_host, out, lse, ws, nws, st));
}

// bind(addresses by name, Problem, _ptr, _ptr_addressable, _stream): where the loaded library has its entry points, and what
// binding.py makes of an argument.
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5 || !PyType_Check(a[1])) {
    PyErr_SetString(PyExc_TypeError, "bind(addresses, Problem, _ptr, _ptr_addressable, _stream)");
    return nullptr;
  }
  PyObject* const d = a[0];
#define SCOUT_BIND(NAME)                                                              \
  do {                                                                                \
    PyObject* o = PyDict_Check(d) ? PyDict_GetItemString(d, #NAME) : nullptr;         \
    void* v = o ? PyLong_AsVoidPtr(o) : nullptr;                                      \
    if (v == nullptr) {                                                               \
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #NAME);                  \
      return nullptr;                                                                 \
    }                                                                                 \
    T.NAME = reinterpret_cast<decltype(T.NAME)>(v);                                   \
  } while (0)
  SCOUT_BIND(build_digests);
  SCOUT_BIND(append_token);
  SCOUT_BIND(score_blocks);
  SCOUT_BIND(select_topk);
  SCOUT_BIND(scout_select_ahead);
  SCOUT_BIND(sparse_decode_attn);
  SCOUT_BIND(sparse_decode_attn_static);
  SCOUT_BIND(scout_attn_partials);
  SCOUT_BIND(scout_attn_finish);
  SCOUT_BIND(merge_partials);
  SCOUT_BIND(periodic_recall);
  SCOUT_BIND(recall_fetch);
  SCOUT_BIND(recall_scatter);
  SCOUT_BIND(scout_layer_step);
  PyObject** const kept[] = {&py.problem, &py.ptr, &py.ptr_addressable, &py.stream};
  for (int i = 0; i < 4; ++i) {
    Py_INCREF(a[i + 1]);
    Py_XSETREF(*kept[i], a[i + 1]);
  }
  Py_RETURN_NONE;
}

// used_by_stream(pinned tensor)
PyObject* py_used_by_stream(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 1 || !THPVariable_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "used_by_stream(tensor)");
    return nullptr;
  }
  used_by_stream(THPVariable_Unpack(a[0]));
  Py_RETURN_NONE;
}

// Nothing that torch throws passes into the interpreter's C frames.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (py.problem == nullptr && F != py_bind) {
    PyErr_SetString(PyExc_RuntimeError, "bind() comes first");
    return nullptr;
  }
  return F(self, a, n);
  END_HANDLE_TH_ERRORS
}

#define SCOUT_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<py_##NAME>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SCOUT_METHOD(bind),
    SCOUT_METHOD(used_by_stream),
    SCOUT_METHOD(build_digests),
    SCOUT_METHOD(append_token),
    SCOUT_METHOD(score_blocks),
    SCOUT_METHOD(select_topk),
    SCOUT_METHOD(select_ahead),
    SCOUT_METHOD(sparse_decode_attn),
    SCOUT_METHOD(sparse_decode_attn_static),
    SCOUT_METHOD(attn_partials),
    SCOUT_METHOD(attn_finish),
    SCOUT_METHOD(attn_finish_ahead),
    SCOUT_METHOD(merge_partials),
    SCOUT_METHOD(periodic_recall),
    SCOUT_METHOD(recall_fetch),
    SCOUT_METHOD(recall_scatter),
    SCOUT_METHOD(layer_step),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
