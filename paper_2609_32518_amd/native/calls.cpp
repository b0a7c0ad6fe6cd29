// The binding's calls in native code: argument checks, output allocation, the current stream and
// the library call of the per-layer and per-chunk entry points, without Python in between.
//
// What bounds the small calls is the host: a step of 72 queries runs 13 us on the GPU, and the
// checks, attribute reads and ctypes conversions of the Python binding took 17.5 us to enqueue it
// (a projection 10.9, a renoise + emit pair 18.4); from here the same calls take a fraction of that.
//
// Each function handles the ordinary call (plain strided CUDA tensors of the shapes, types and
// strides the kernels assume, the current stream) and returns its result.  For anything else it
// returns None before the library's call, and the caller's Python path, which checks everything again,
// handles the call or raises.  Once the library's call has been made nothing goes back to that path:
// kernels of a call that reports an error may be on the stream already, and run again an update in
// place would be applied twice.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <exception>
#include <memory>

#include "unstep.h"

namespace {

constexpr int64_t kD = UNSTEP_HEAD_DIM;
constexpr const char* kCapsule = "unstep.Cache";

// What the calls need of a Cache object (the handle stays owned by it).
struct CacheInfo {
  unstep_cache* handle;
  int64_t B, H, T;
  c10::Device device;
  PyObject* scratch_methods;    // the tuple (Cache.workspace, Cache.workspace_bytes, Cache._step_workspace)
  ~CacheInfo() { Py_XDECREF(scratch_methods); }
};

// A plain strided tensor on a GPU: exactly torch.Tensor or Parameter, no subclass, no functorch
// wrapper, no fake or tracing tensor.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || at::isTensorSubclassLike(t) || t.is_neg())
    return nullptr;
  return &t;
}

bool usable(const at::Tensor& t) { return t.defined() && t.is_cuda() && !at::isTensorSubclassLike(t) && t.has_storage(); }

bool is(const at::Tensor* t, at::ScalarType type, at::IntArrayRef shape, c10::Device dev) {
  return t && t->scalar_type() == type && t->sizes() == shape && t->device() == dev && t->is_contiguous();
}

bool to_i32(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  if (over || x < INT32_MIN || x > INT32_MAX) return false;
  *v = int32_t(x);
  return true;
}

bool to_f64(PyObject* o, double* v) {
  if (!PyFloat_CheckExact(o)) return false;
  *v = PyFloat_AS_DOUBLE(o);
  return true;
}

void* current_stream() { return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

const CacheInfo* cache_of(PyObject* o) { return static_cast<const CacheInfo*>(PyCapsule_GetPointer(o, kCapsule)); }

PyObject* none() {
  PyErr_Clear();
  Py_RETURN_NONE;
}

// A Python reference owned here.
struct Ref {
  PyObject* o;
  explicit Ref(PyObject* x) : o(x) {}
  Ref(const Ref&) = delete;
  ~Ref() { Py_XDECREF(o); }
  PyObject* release() {
    PyObject* r = o;
    o = nullptr;
    return r;
  }
};

// Sets the package's UnstepError(rc, message) for the library's last error on this thread.
void raise(int rc) {
  const Ref pkg{PyImport_ImportModule("paper_2609_32518_amd")};
  const Ref type{pkg.o ? PyObject_GetAttrString(pkg.o, "UnstepError") : nullptr};
  const Ref err{type.o ? PyObject_CallFunction(type.o, "is", rc, unstep_last_error()) : nullptr};
  if (err.o) PyErr_SetObject(type.o, err.o);
}

// Runs the library call without the GIL; on an error of the library false, with that error raised.
// A tensor's data_ptr may throw (a storage without memory), so the pointers are read before this: an
// exception must not leave a region without the GIL.
template <class F>
bool call(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = f();
  Py_END_ALLOW_THREADS;
  if (rc != UNSTEP_OK) raise(rc);
  return rc == UNSTEP_OK;
}

// No C++ exception leaves a function of the module.
template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const std::exception&) {
    return none();
  }
}

at::Tensor new_bf16(at::IntArrayRef shape, c10::Device dev) {
  return at::empty(shape, at::TensorOptions().dtype(at::kBFloat16).device(dev));
}

// q, k, v of a chunk: [B, N, H, 128] bf16, unit stride on the last axis, batch stride N * token
// stride, one (token, head) stride pair for all.
struct Chunk {
  int32_t f0, C;
  int64_t N;
  const at::Tensor *q, *k, *v, *cos, *sin;
  int64_t ts, hs;
  const void *qp, *kp, *vp;
  const float *cp, *sp;
};

void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

bool chunk_of(const CacheInfo& c, PyObject* const* a, bool q_optional, Chunk* o) {
  if (!to_i32(a[0], &o->f0) || !to_i32(a[1], &o->C) || o->C < 1) return false;
  o->N = int64_t(o->C) * c.T;
  const int64_t shape[4] = {c.B, o->N, c.H, kD};
  o->q = nullptr;
  if (a[2] != Py_None || !q_optional) {
    if (!(o->q = plain(a[2]))) return false;
  }
  if (!(o->k = plain(a[3])) || !(o->v = plain(a[4]))) return false;
  o->ts = o->hs = -1;
  for (const at::Tensor* t : {o->k, o->v, o->q}) {
    if (!t) continue;
    if (t->scalar_type() != at::kBFloat16 || t->sizes() != at::IntArrayRef(shape, 4) || t->device() != c.device) return false;
    if (t->stride(3) != 1 || (c.B > 1 && t->stride(0) != o->N * t->stride(1))) return false;
    if (t == o->k) {
      o->ts = t->stride(1);
      o->hs = t->stride(2);
    } else if (t->stride(1) != o->ts || t->stride(2) != o->hs) {
      return false;
    }
  }
  const int64_t tab[2] = {o->N, kD / 2};
  o->cos = plain(a[5]);
  o->sin = plain(a[6]);
  if (!is(o->cos, at::kFloat, at::IntArrayRef(tab, 2), c.device) || !is(o->sin, at::kFloat, at::IntArrayRef(tab, 2), c.device))
    return false;
  o->qp = ptr(o->q);
  o->kp = ptr(o->k);
  o->vp = ptr(o->v);
  o->cp = static_cast<const float*>(ptr(o->cos));
  o->sp = static_cast<const float*>(ptr(o->sin));
  return true;
}

// A given [B, N, H, 128] output checked, or a new one in *made.
const at::Tensor* chunk_out(const CacheInfo& c, int64_t N, PyObject* o, at::Tensor* made) {
  const int64_t shape[4] = {c.B, N, c.H, kD};
  if (o == Py_None) {
    *made = new_bf16(at::IntArrayRef(shape, 4), c.device);
    return usable(*made) ? made : nullptr;
  }
  const at::Tensor* t = plain(o);
  return is(t, at::kBFloat16, at::IntArrayRef(shape, 4), c.device) ? t : nullptr;
}

// The object that a call returns, made before the library's call (null, with a Python error, if that
// fails).
Ref result(PyObject* given, const at::Tensor& made) {
  if (given != Py_None) {
    Py_INCREF(given);
    return Ref{given};
  }
  return Ref{THPVariable_Wrap(made)};
}

// What the appends return: a tuple of the rotated queries, or of None without queries.
Ref append_result(bool with_q, PyObject* given, const at::Tensor& made) {
  if (!with_q) return Ref{Py_BuildValue("(O)", Py_None)};
  Ref r = result(given, made);
  return Ref{r.o ? Py_BuildValue("(N)", r.release()) : nullptr};
}

// lse: None or fp32 [B, H, N]
bool lse_of(const CacheInfo& c, int64_t N, PyObject* o, float** p) {
  *p = nullptr;
  if (o == Py_None) return true;
  const int64_t shape[3] = {c.B, c.H, N};
  const at::Tensor* t = plain(o);
  if (!is(t, at::kFloat, at::IntArrayRef(shape, 3), c.device)) return false;
  *p = static_cast<float*>(ptr(t));
  return true;
}

// Whether the scratch methods that a call would ask (`step`: _step_workspace too) are the binding's own on
// `owner`: a subclass, or a program that replaced one, is asked through the Python path.
PyObject* scratch_names[3];    // interned, made with the module
bool own_scratch(const CacheInfo& c, PyObject* owner, bool step) {
  for (int i = 0; i < (step ? 3 : 2); ++i) {
    const Ref m{PyObject_GetAttr(owner, scratch_names[i])};
    if (!m.o || !PyMethod_Check(m.o) || PyMethod_GET_FUNCTION(m.o) != PyTuple_GET_ITEM(c.scratch_methods, i) ||
        PyMethod_GET_SELF(m.o) != owner)
      return false;
  }
  return true;
}

// The split-key scratch: the given tensor, or (use_split) the one the Cache object keeps as _ws,
// replaced by a larger one when it is too small, as Cache.workspace does.  The kept tensor is held in
// *hold until the call has been enqueued.
bool workspace_of(const CacheInfo& c, int32_t f0, int32_t C, int32_t W, PyObject* given, PyObject* use_split, PyObject* owner,
                  bool step, at::Tensor* hold, void** p, size_t* bytes) {
  *p = nullptr;
  *bytes = 0;
  if (given != Py_None) {
    const at::Tensor* t = plain(given);
    if (!t || t->device() != c.device || !t->is_contiguous()) return false;
    *p = t->data_ptr();
    *bytes = size_t(t->numel()) * t->element_size();
    return true;
  }
  if (use_split == Py_False) return true;
  if (use_split != Py_True || !own_scratch(c, owner, step)) return false;
  size_t need = 0;
  if (unstep_attn_workspace_size(c.handle, f0, C, W, &need) != UNSTEP_OK) return false;
  if (need == 0) return true;
  const Ref kept{PyObject_GetAttrString(owner, "_ws")};
  if (!kept.o) return false;
  const at::Tensor* t = kept.o == Py_None ? nullptr : plain(kept.o);
  if (kept.o != Py_None && !t) return false;
  if (t && size_t(t->numel()) >= need) {
    *hold = *t;
  } else {
    *hold = at::empty({int64_t(need)}, at::TensorOptions().dtype(at::kByte).device(c.device));
    if (!usable(*hold)) return false;
    const Ref made{THPVariable_Wrap(*hold)};
    if (!made.o || PyObject_SetAttrString(owner, "_ws", made.o) != 0) return false;
  }
  *p = hold->data_ptr();
  *bytes = size_t(hold->numel());
  return true;
}

// ---- functions ------------------------------------------------------------------------------------

// cache(handle, B, H, T, k, scratch_methods) -> capsule
PyObject* f_cache(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const at::Tensor* k = n == 6 ? plain(a[4]) : nullptr;
    if (!k || !PyTuple_CheckExact(a[5]) || PyTuple_GET_SIZE(a[5]) != 3) return none();
    auto info = std::unique_ptr<CacheInfo>(new CacheInfo{static_cast<unstep_cache*>(PyLong_AsVoidPtr(a[0])), PyLong_AsLongLong(a[1]),
                                                         PyLong_AsLongLong(a[2]), PyLong_AsLongLong(a[3]), k->device(),
                                                         (Py_INCREF(a[5]), a[5])});
    if (PyErr_Occurred()) return none();
    PyObject* cap = PyCapsule_New(info.get(), kCapsule, [](PyObject* o) {
      delete static_cast<CacheInfo*>(PyCapsule_GetPointer(o, kCapsule));
    });
    if (cap) info.release();
    return cap;
  });
}

// append(cache, f0, C, q, k, v, cos, sin, q_rot) -> (q_rot or None,)
PyObject* f_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const CacheInfo* c = n == 9 ? cache_of(a[0]) : nullptr;
    Chunk k;
    if (!c || !chunk_of(*c, a + 1, true, &k)) return none();
    at::Tensor made;
    const at::Tensor* qr = nullptr;
    if (k.q && !(qr = chunk_out(*c, k.N, a[8], &made))) return none();
    if (!k.q && a[8] != Py_None) return none();
    Ref r = append_result(k.q != nullptr, a[8], made);
    if (!r.o) return none();
    void *st = current_stream(), *qrp = ptr(qr);
    if (!call([&] { return unstep_kv_append(c->handle, k.f0, k.C, k.qp, k.kp, k.vp, k.ts, k.hs, k.cp, k.sp, qrp, st); }))
      return nullptr;
    return r.release();
  });
}

// append_qknorm(cache, f0, C, q, k, v, cos, sin, wq, wk, eps, q_rot) -> (q_rot or None,)
PyObject* f_append_qknorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const CacheInfo* c = n == 12 ? cache_of(a[0]) : nullptr;
    Chunk k;
    double eps;
    if (!c || !chunk_of(*c, a + 1, true, &k) || !to_f64(a[10], &eps)) return none();
    const int64_t shape[1] = {c->H * kD};
    const at::Tensor *wk = plain(a[9]), *wq = k.q ? plain(a[8]) : nullptr;
    if (!is(wk, at::kBFloat16, at::IntArrayRef(shape, 1), c->device)) return none();
    at::Tensor made;
    const at::Tensor* qr = nullptr;
    if (k.q) {
      if (!is(wq, at::kBFloat16, at::IntArrayRef(shape, 1), c->device) || !(qr = chunk_out(*c, k.N, a[11], &made))) return none();
    } else if (a[8] != Py_None || a[11] != Py_None) {
      return none();
    }
    Ref r = append_result(k.q != nullptr, a[11], made);
    if (!r.o) return none();
    void *st = current_stream(), *qrp = ptr(qr), *wqp = ptr(wq), *wkp = ptr(wk);
    if (!call([&] {
          return unstep_kv_append_qknorm(c->handle, k.f0, k.C, k.qp, k.kp, k.vp, k.ts, k.hs, k.cp, k.sp, wqp, wkp, eps, qrp, st);
        }))
      return nullptr;
    return r.release();
  });
}

// window_attn(cache, f0, C, W, q_rot, out, lse, scale, workspace, use_split, owner) -> out
PyObject* f_window_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const CacheInfo* c = n == 11 ? cache_of(a[0]) : nullptr;
    int32_t f0, C, W;
    double scale;
    if (!c || !to_i32(a[1], &f0) || !to_i32(a[2], &C) || C < 1 || !to_i32(a[3], &W) || !to_f64(a[7], &scale)) return none();
    const int64_t N = int64_t(C) * c->T;
    const int64_t shape[4] = {c->B, N, c->H, kD};
    const at::Tensor* q = plain(a[4]);
    float* lse;
    void* ws;
    size_t bytes;
    at::Tensor made, hold;
    if (!is(q, at::kBFloat16, at::IntArrayRef(shape, 4), c->device) || !lse_of(*c, N, a[6], &lse) ||
        !workspace_of(*c, f0, C, W, a[8], a[9], a[10], false, &hold, &ws, &bytes))
      return none();
    const at::Tensor* out = chunk_out(*c, N, a[5], &made);
    if (!out) return none();
    Ref r = result(a[5], made);
    if (!r.o) return none();
    void *st = current_stream(), *qp = ptr(q), *op = ptr(out);
    if (!call([&] { return unstep_window_attn(c->handle, f0, C, W, qp, op, lse, float(scale), ws, bytes, st); }))
      return nullptr;
    return r.release();
  });
}

// step(cache, f0, C, q, k, v, cos, sin, W, q_rot, out, lse, scale, workspace, use_split, owner) -> out
PyObject* f_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const CacheInfo* c = n == 16 ? cache_of(a[0]) : nullptr;
    Chunk k;
    int32_t W;
    double scale;
    float* lse;
    void* ws;
    size_t bytes;
    at::Tensor hold;
    if (!c || !chunk_of(*c, a + 1, false, &k) || !to_i32(a[8], &W) || !to_f64(a[12], &scale) || !lse_of(*c, k.N, a[11], &lse) ||
        !workspace_of(*c, k.f0, k.C, W, a[13], a[14], a[15], true, &hold, &ws, &bytes))
      return none();
    at::Tensor made_q, made;
    const at::Tensor *qr = chunk_out(*c, k.N, a[9], &made_q), *out = qr ? chunk_out(*c, k.N, a[10], &made) : nullptr;
    if (!out) return none();
    Ref r = result(a[10], made);
    if (!r.o) return none();
    void *st = current_stream(), *qrp = ptr(qr), *op = ptr(out);
    if (!call([&] {
          return unstep_step(c->handle, k.f0, k.C, W, k.qp, k.kp, k.vp, k.ts, k.hs, k.cp, k.sp, qrp, op, lse, float(scale), ws, bytes,
                             st);
        }))
      return nullptr;
    return r.release();
  });
}

// linear(x, w, bias, out) -> out
PyObject* f_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 4) return none();
    const at::Tensor *x = plain(a[0]), *w = plain(a[1]), *b = a[2] == Py_None ? nullptr : plain(a[2]);
    if (!x || !w || (a[2] != Py_None && !b)) return none();
    for (const at::Tensor* t : {x, w, b})
      if (t && (t->scalar_type() != at::kBFloat16 || !t->is_contiguous() || t->device() != x->device())) return none();
    if (w->dim() != 2 || x->dim() < 1) return none();
    const int64_t N = w->size(0), K = w->size(1);
    if (K < 1 || x->size(-1) != K || (b && (b->dim() != 1 || b->size(0) != N))) return none();
    const int64_t M = x->numel() / K;
    if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return none();
    at::DimVector shape(x->sizes().begin(), x->sizes().end());
    shape.back() = N;
    at::Tensor made;
    const at::Tensor* out = &made;
    if (a[3] == Py_None) {
      made = new_bf16(shape, x->device());
      if (!usable(made)) return none();
    } else if (!is(out = plain(a[3]), at::kBFloat16, shape, x->device())) {
      return none();
    }
    Ref r = result(a[3], made);
    if (!r.o) return none();
    void *st = current_stream(), *xp = ptr(x), *wp = ptr(w), *bp = ptr(b), *op = ptr(out);
    if (!call([&] { return unstep_linear(xp, wp, bp, op, int32_t(M), int32_t(N), int32_t(K), st); }))
      return nullptr;
    return r.release();
  });
}

// flow(emit, x, y, sigma, out) -> out: the renoise (emit False) or emit (True) update
PyObject* f_flow(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    double sigma;
    if (n != 5 || !to_f64(a[3], &sigma)) return none();
    const at::Tensor *x = plain(a[1]), *y = plain(a[2]);
    if (!x || !y) return none();
    for (const at::Tensor* t : {x, y})
      if (t->scalar_type() != at::kBFloat16 || !t->is_contiguous() || t->device() != x->device()) return none();
    if (x->sizes() != y->sizes()) return none();
    at::Tensor made;
    const at::Tensor* out = &made;
    if (a[4] == Py_None) {
      made = new_bf16(x->sizes(), x->device());
      if (!usable(made)) return none();
    } else if (!is(out = plain(a[4]), at::kBFloat16, x->sizes(), x->device())) {
      return none();
    }
    const bool emit = a[0] == Py_True;
    const int64_t count = x->numel();
    Ref r = result(a[4], made);
    if (!r.o) return none();
    void *st = current_stream(), *xp = ptr(x), *yp = ptr(y), *op = ptr(out);
    if (!call([&] { return emit ? unstep_emit(xp, yp, sigma, op, count, st) : unstep_renoise(xp, yp, sigma, op, count, st); }))
      return nullptr;
    return r.release();
  });
}

#define UNSTEP_FN(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {UNSTEP_FN(cache), UNSTEP_FN(append), UNSTEP_FN(append_qknorm), UNSTEP_FN(window_attn),
                         UNSTEP_FN(step),  UNSTEP_FN(linear), UNSTEP_FN(flow),          {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  const char* const names[3] = {"workspace", "workspace_bytes", "_step_workspace"};
  for (int i = 0; i < 3; ++i)
    if (!(scratch_names[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
  return PyModule_Create(&module);
}
